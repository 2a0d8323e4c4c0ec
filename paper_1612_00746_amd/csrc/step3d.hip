// Observables of three particles on a chain (the propagation is in
// step3c.hip): the ensemble's two-body marginals in FP64 and the occupation
// and pair correlation from them.
//
// One pass over the state: a block holds 32 x2 rows by 128 x3 columns (8 rows
// and two columns per lane and wave) and runs over a chunk of x1 planes, at
// each plane over a segment of the realisations (p = |psi|^2 only ever enters
// as a sum over them).  The sum over x3 is reduced across the wave and the
// sum over x2 across the block once per plane; the sum over x1 stays in
// registers.  Bound by reading the state: 64 x 256^3 complex64, 8.6 GB,
// 1.46 ms, 5.9 TB/s (one launch for the x3 sums and one for the others took
// 4.6 ms).
#include "ctqw_internal.hpp"
#include "wave_sum.hpp"

namespace ctqw {
namespace {

constexpr int kRows3 = 8;                // x2 rows per wave
constexpr int kTile2 = 4 * kRows3;       // x2 rows of a block
constexpr int kTile3 = 128;              // x3 columns

template <typename C>
__global__ void __launch_bounds__(256) marg3_kernel(Obs3Args a) {
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int N = a.max_N;
    const int64_t NN = (int64_t)N * N;
    int b = (int)blockIdx.x;
    const int p3 = b % a.panels;
    b /= a.panels;
    const int p2 = b % a.chunks;
    b /= a.chunks;
    const int px = b % a.planes;
    const int seg = b / a.planes;
    const int x2 = p2 * kTile2 + wv * kRows3, x3 = p3 * kTile3 + lane;
    const int xa = (int)((int64_t)N * px / a.planes), xb = (int)((int64_t)N * (px + 1) / a.planes);
    const int64_t ra = a.R * seg / a.segs, rb = a.R * (seg + 1) / a.segs;
    using F64 = const __attribute__((address_space(4))) double*;

    double s23[kRows3][2];
    int at[kRows3][2];
    bool on[kRows3][2];
#pragma unroll
    for (int i = 0; i < kRows3; ++i)
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            s23[i][p] = 0.0;
            // (off the lattice: the tile's first element, with weight 0, so that
            // all loads of a row group are issued without branches)
            on[i][p] = x2 + i < N && x3 + 64 * p < N;
            at[i][p] = on[i][p] ? (x2 + i) * N + x3 + 64 * p : 0;
        }
    double* const M12 = a.M + (int64_t)(seg * a.panels + p3) * NN;
    double* const M13 = a.M + a.off13 + (int64_t)(seg * a.chunks + p2) * NN;
    double* const M23 = a.M + a.off23 + (int64_t)(seg * a.planes + px) * NN;
    __shared__ double cols[2][4][kTile3];
    for (int x1 = xa; x1 < xb; ++x1) {
        double t[kRows3][2];
#pragma unroll
        for (int i = 0; i < kRows3; ++i) t[i][0] = t[i][1] = 0.0;
        for (int64_t r = ra; r < rb; ++r) {
            const C* psi = reinterpret_cast<const C*>(a.psi) + (r * N + x1) * NN;
            const double sc = ((F64)a.scale)[r];
            const double w = sc * sc;
            C v[kRows3][2];
#pragma unroll
            for (int i = 0; i < kRows3; ++i)
#pragma unroll
                for (int p = 0; p < 2; ++p) v[i][p] = psi[at[i][p]];
#pragma unroll
            for (int i = 0; i < kRows3; ++i)
#pragma unroll
                for (int p = 0; p < 2; ++p) {
                    const double re = v[i][p].x, im = v[i][p].y;
                    const double s = __builtin_fma(w, __builtin_fma(im, im, re * re), t[i][p]);
                    t[i][p] = on[i][p] ? s : 0.0;
                }
        }
        double c0 = 0.0, c1 = 0.0;
#pragma unroll
        for (int i = 0; i < kRows3; ++i) {
            s23[i][0] += t[i][0];
            s23[i][1] += t[i][1];
            c0 += t[i][0];
            c1 += t[i][1];
            const double s = wave_sum_last(t[i][0] + t[i][1]);
            if (lane == 63 && x2 + i < N) M12[(int64_t)x1 * N + x2 + i] = s;
        }
        double(*const cb)[kTile3] = cols[x1 & 1];   // two sets: one barrier per plane
        cb[wv][lane] = c0;
        cb[wv][lane + 64] = c1;
        __syncthreads();
        if (threadIdx.x < kTile3 && p3 * kTile3 + (int)threadIdx.x < N) {
            const int k = threadIdx.x;
            M13[(int64_t)x1 * N + p3 * kTile3 + k] = ((cb[0][k] + cb[1][k]) + cb[2][k]) + cb[3][k];
        }
    }
#pragma unroll
    for (int i = 0; i < kRows3; ++i)
#pragma unroll
        for (int p = 0; p < 2; ++p)
            if (on[i][p]) M23[at[i][p]] = s23[i][p];
}

// E[0..2] = the ensemble's M12, M13, M23: the blocks' partials in order.
__global__ void marg3_sum_kernel(Obs3Args a) {
    const int64_t NN = (int64_t)a.max_N * a.max_N;
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= NN) return;
    const int which = blockIdx.y;
    const int n = a.segs * (which == 0 ? a.panels : (which == 1 ? a.chunks : a.planes));
    const double* src = a.M + (which == 0 ? 0 : (which == 1 ? a.off13 : a.off23)) + e;
    double s = 0.0;
#pragma unroll 8
    for (int k = 0; k < n; ++k) s += src[k * NN];
    a.E[which * NN + e] = s / (double)a.R;
}

// occupation n(i) = sum_j E12[i][j] + E12[j][i] + E13[j][i]; pair G(i, j) =
// E12 + E12^T + E13 + E13^T + E23 + E23^T at (i, j).  A block per node i.
__global__ void __launch_bounds__(256) obs3_ensemble_kernel(Obs3Args a) {
    const int N = a.max_N, i = blockIdx.x;
    const int64_t NN = (int64_t)N * N;
    const double* E12 = a.E;
    const double* E13 = a.E + NN;
    const double* E23 = a.E + 2 * NN;
    __shared__ double sum[256];
    double occ = 0.0;
    for (int j = threadIdx.x; j < N; j += 256) {
        const int64_t ij = (int64_t)i * N + j, ji = (int64_t)j * N + i;
        const double both = E12[ij] + E12[ji], m13 = E13[ji];
        occ += both + m13;
        if (a.want_pair) a.out[N + ij] = both + (E13[ij] + m13) + (E23[ij] + E23[ji]);
    }
    sum[threadIdx.x] = occ;
    __syncthreads();
    for (int h = 128; h >= 1; h >>= 1) {
        if ((int)threadIdx.x < h) sum[threadIdx.x] += sum[threadIdx.x + h];
        __syncthreads();
    }
    if (threadIdx.x == 0) a.out[i] = sum[0];
}

}  // namespace

// Blocks: x1 in chunks of planes, then the realisations in segments, until
// the launch has four blocks per compute unit.
void obs3_split(int N, int64_t R, Obs3Args* a) {
    constexpr int64_t kBlocks = 1024;
    a->panels = (N + kTile3 - 1) / kTile3;
    a->chunks = (N + kTile2 - 1) / kTile2;
    const int64_t tiles = (int64_t)a->panels * a->chunks;
    a->planes = (int32_t)std::max<int64_t>(1, std::min<int64_t>(N, (kBlocks + tiles - 1) / tiles));
    a->segs = (int32_t)std::max<int64_t>(1, std::min<int64_t>(R, kBlocks / (tiles * a->planes)));
    const int64_t NN = (int64_t)N * N;
    a->off13 = (int64_t)a->segs * a->panels * NN;
    a->off23 = a->off13 + (int64_t)a->segs * a->chunks * NN;
    a->partials = a->off23 + (int64_t)a->segs * a->planes * NN;
}

hipError_t launch_obs3(const Obs3Args& a, int dtype, hipStream_t s) {
    const int N = a.max_N;
    const int64_t blocks = (int64_t)a.panels * a.chunks * a.planes * a.segs;
    if (blocks < 1 || blocks > INT32_MAX) return hipErrorInvalidValue;
    if (dtype == 1) hipLaunchKernelGGL(marg3_kernel<double2>, dim3((unsigned)blocks), dim3(256), 0, s, a);
    else hipLaunchKernelGGL(marg3_kernel<float2>, dim3((unsigned)blocks), dim3(256), 0, s, a);
    const int64_t NN = (int64_t)N * N;
    hipLaunchKernelGGL(marg3_sum_kernel, dim3((unsigned)((NN + 255) / 256), 3), dim3(256), 0, s, a);
    hipLaunchKernelGGL(obs3_ensemble_kernel, dim3((unsigned)N), dim3(256), 0, s, a);
    return hipGetLastError();
}

}  // namespace ctqw
