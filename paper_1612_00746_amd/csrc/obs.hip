// Ensemble observables of one and two particles: occupation and pair
// correlation from the diagonal of the ensemble-averaged density matrix
// (Eq. 2 and the post-processing of Algs. 1-3).
//
// Both are sums over realisations of p = |psi|^2, so one pass over the state
// adds p up at fixed (x1, x2) over a group's realisations and reduces the
// sums to rows and columns once per tile, not once per realisation:
//   obs_tile_kernel  a block holds a tile of 16 x 128 pairs of one group and
//                    runs over a segment of its realisations (as many
//                    segments as fill the device), FP64 in registers;
//   obs_occ_kernel   adds the tiles' row and column sums in a fixed order;
//   obs_pair_kernel  adds the segments' tiles and their mirror images.
// It reads each amplitude once and is bound by that: 4096 realisations of 64
// to 1024 nodes, 12.2 GB, 1.99 ms, 6.2 TB/s (a pass for the columns and one for the rows
// took 5.94 ms); 1000 x two bosons N = 128 complex128 with pairs 0.11 ms, where
// a thread per site and per pair adding up 1000 realisations took 1.48 ms.
// One particle: the tile's rows are realisations.
#include "ctqw_internal.hpp"
#include "wave_sum.hpp"

namespace ctqw {
namespace {

constexpr int kRows = 16;       // rows of a tile: 4 waves x 4
constexpr int kCols = 128;      // columns: two per lane, 64 apart
constexpr int kPerWave = kRows / 4;

template <typename S>
__device__ __forceinline__ S uniform_entry(const S* table, int index) {
    using P = const __attribute__((address_space(4))) int32_t*;
    S v;
    const P src = (P)(table + index);
    int32_t* dst = reinterpret_cast<int32_t*>(&v);
#pragma unroll
    for (int k = 0; k < (int)(sizeof(S) / 4); ++k) dst[k] = src[k];
    return v;
}

// The group whose blocks hold block b (blocks of a group are consecutive).
__device__ __forceinline__ int group_of(const ObsGroup* groups, int G, int b) {
    int lo = 0, hi = G - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) / 2;
        if (((const __attribute__((address_space(4))) ObsGroup*)groups)[mid].block0 <= b) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

template <typename C, bool ONE>
__global__ void __launch_bounds__(256) obs_tile_kernel(ObsArgs a) {
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const ObsGroup g = uniform_entry(a.groups, group_of(a.groups, a.G, (int)blockIdx.x));
    const int N = g.N;
    int b = (int)blockIdx.x - g.block0;
    const int panel = b % g.panels;
    b /= g.panels;
    const int chunk = b % g.chunks;
    const int seg = b / g.chunks;
    const int c0 = panel * kCols, q0 = chunk * kRows + wv * kPerWave;
    const int Rg = g.last - g.first;
    const int k0 = g.first + (int)((int64_t)Rg * seg / g.segs), k1 = g.first + (int)((int64_t)Rg * (seg + 1) / g.segs);
    const bool tri = !ONE && a.triangle;
    const C* psi = reinterpret_cast<const C*>(a.psi);
    using U32 = const __attribute__((address_space(4))) int32_t*;
    using U64 = const __attribute__((address_space(4))) int64_t*;
    using F64 = const __attribute__((address_space(4))) double*;

    double acc[kPerWave][2];
#pragma unroll
    for (int i = 0; i < kPerWave; ++i) acc[i][0] = acc[i][1] = 0.0;
    // element of row slot i, column p of a realisation (ONE: the rows are
    // realisations); off the grid the first element, with weight 0, so that
    // all loads are issued without branches
    int at[kPerWave][2];
    bool in[kPerWave][2];
    bool any = false;
#pragma unroll
    for (int i = 0; i < kPerWave; ++i)
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            const int q = ONE ? 0 : q0 + i, c = c0 + lane + 64 * p;
            const bool on = c < N && q < N && (!tri || c >= q);
            in[i][p] = on;
            at[i][p] = on ? (tri ? q * N - (q * (q + 1)) / 2 + c : q * N + c) : 0;
            any = any || on;
        }
    // (a wave whose rows lie wholly below the diagonal, or past the grid)
    if (ONE || __builtin_amdgcn_ballot_w64(any) != 0) {
        const int step = ONE ? kRows : 1;
#pragma unroll 2
        for (int k = k0; k < k1; k += step) {
            C v[kPerWave][2];
            double w[kPerWave];
#pragma unroll
            for (int i = 0; i < kPerWave; ++i) {
                const int kk = ONE ? min(k + wv * kPerWave + i, k1 - 1) : k;
                const int r = ((U32)a.group_members)[kk];
                const int64_t off = ((U64)(a.reals + r))[0];   // RealDev::state_off
                const double sc = ((F64)a.scale)[r];
                w[i] = sc * sc;
#pragma unroll
                for (int p = 0; p < 2; ++p) v[i][p] = psi[off + at[i][p]];
            }
#pragma unroll
            for (int i = 0; i < kPerWave; ++i) {
                const bool live = !ONE || k + wv * kPerWave + i < k1;
#pragma unroll
                for (int p = 0; p < 2; ++p) {
                    const double re = v[i][p].x, im = v[i][p].y;
                    const double s = __builtin_fma(w[i], __builtin_fma(im, im, re * re), acc[i][p]);
                    acc[i][p] = live && in[i][p] ? s : acc[i][p];
                }
            }
        }
    }
    // Pairs: the tile's sums over this segment.
    if (!ONE && a.want_pair) {
        double* pp = a.pair_part + g.pair_off + (int64_t)seg * N * N;
#pragma unroll
        for (int i = 0; i < kPerWave; ++i)
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                const int q = q0 + i, c = c0 + lane + 64 * p;
                if (q < N && c < N) pp[(int64_t)q * N + c] = acc[i][p];
            }
    }
    // n_i adds row i and column i; the triangle stores a pair once (weight 2 to
    // both its nodes; a doubly occupied node counts 2, given to its row).
    __shared__ double cols[4][kCols];
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        double s = 0.0;
#pragma unroll
        for (int i = 0; i < kPerWave; ++i) {
            const double w = tri ? (c0 + lane + 64 * p == q0 + i ? 0.0 : 2.0) : 1.0;
            s = __builtin_fma(w, acc[i][p], s);
        }
        cols[wv][lane + 64 * p] = s;
    }
    if constexpr (!ONE) {
#pragma unroll
        for (int i = 0; i < kPerWave; ++i) {
            const double s = wave_sum_last(acc[i][0] + acc[i][1]);
            if (lane == 63 && q0 + i < N)
                a.row_part[g.row_off + ((int64_t)seg * g.panels + panel) * N + q0 + i] = tri ? 2.0 * s : s;
        }
    }
    __syncthreads();
    if (threadIdx.x < kCols && c0 + (int)threadIdx.x < N) {
        const int t = threadIdx.x;
        a.col_part[g.col_off + ((int64_t)seg * g.chunks + chunk) * N + c0 + t] =
            ((cols[0][t] + cols[1][t]) + cols[2][t]) + cols[3][t];
    }
}

// Occupation of 64 sites of a group: 16 waves add the tiles' partials (wave
// w those at w, w + 16, ...), then one adds the waves' sums.
__global__ void __launch_bounds__(1024) obs_occ_kernel(ObsArgs a) {
    const ObsGroup g = uniform_entry(a.groups, (int)blockIdx.y);
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int i = blockIdx.x * 64 + lane;
    __shared__ double sum[16][64];
    double s = 0.0;
    if (i < g.N) {
        const int nr = a.m == 1 ? 0 : g.segs * g.panels, nc = g.segs * g.chunks;
        const double* rp = a.row_part + g.row_off + i;
        const double* cp = a.col_part + g.col_off + i;
#pragma unroll 4
        for (int k = wv; k < nr; k += 16) s += rp[(int64_t)k * g.N];
#pragma unroll 4
        for (int k = wv; k < nc; k += 16) s += cp[(int64_t)k * g.N];
    }
    sum[wv][lane] = s;
    __syncthreads();
    if (wv == 0 && i < g.N) {
        double t = 0.0;
#pragma unroll
        for (int w = 0; w < 16; ++w) t += sum[w][lane];
        a.out[g.out_off + i] = t / (double)(g.last - g.first);
    }
}

// Pair correlation G(i, j) = p(i, j) + p(j, i) (triangle: 2 p of the stored
// pair), 32 x 32 entries per block; the segments are added in order.
__global__ void __launch_bounds__(256) obs_pair_kernel(ObsArgs a) {
    const ObsGroup g = uniform_entry(a.groups, (int)blockIdx.z);
    const int N = g.N;
    const int i0 = blockIdx.y * 32, j0 = blockIdx.x * 32;
    if (i0 >= N || j0 >= N) return;   // block-uniform
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
    __shared__ double mirror[32][33];
    const double* pp = a.pair_part + g.pair_off;
    const int64_t NN = (int64_t)N * N;
    auto total = [&](int q, int c) {
        double s = 0.0;
        if (q < N && c < N && (!a.triangle || c >= q)) {
            const double* e = pp + (int64_t)q * N + c;
#pragma unroll 4
            for (int k = 0; k < g.segs; ++k) s += e[k * NN];
        }
        return s;
    };
    for (int y = ty; y < 32; y += 8) mirror[y][tx] = total(j0 + y, i0 + tx);
    __syncthreads();
    for (int y = ty; y < 32; y += 8) {
        const int i = i0 + y, j = j0 + tx;
        if (i >= N || j >= N) continue;
        const double direct = total(i, j), other = mirror[tx][y];
        const double s = a.triangle && i == j ? 2.0 * direct : (a.triangle ? 2.0 * (direct + other) : direct + other);
        a.out[g.out_off + N + (int64_t)i * N + j] = s / (double)(g.last - g.first);
    }
}

}  // namespace

// Tiles of a lattice of N nodes, and the segments of realisations that give
// the device about kObsBlocks blocks (four per compute unit).
void obs_tiles(int m, int N, int32_t* panels, int32_t* chunks) {
    *panels = (N + kCols - 1) / kCols;
    *chunks = m == 1 ? 1 : (N + kRows - 1) / kRows;
}
int obs_rows_per_pass(int m) { return m == 1 ? kRows : 1; }

hipError_t launch_observables(const ObsArgs& a, hipStream_t stream) {
    if (a.G > 65535 || a.max_N > 65535 || a.blocks < 1) return hipErrorInvalidValue;
    const dim3 gt((unsigned)a.blocks);
    if (a.m == 1) {
        if (a.dtype == 1) hipLaunchKernelGGL((obs_tile_kernel<double2, true>), gt, dim3(256), 0, stream, a);
        else hipLaunchKernelGGL((obs_tile_kernel<float2, true>), gt, dim3(256), 0, stream, a);
    } else {
        if (a.dtype == 1) hipLaunchKernelGGL((obs_tile_kernel<double2, false>), gt, dim3(256), 0, stream, a);
        else hipLaunchKernelGGL((obs_tile_kernel<float2, false>), gt, dim3(256), 0, stream, a);
    }
    hipLaunchKernelGGL(obs_occ_kernel, dim3((a.max_N + 63) / 64, (unsigned)a.G), dim3(1024), 0, stream, a);
    if (a.want_pair && a.m > 1) {
        const unsigned t = (a.max_N + 31) / 32;
        hipLaunchKernelGGL(obs_pair_kernel, dim3(t, t, (unsigned)a.G), dim3(256), 0, stream, a);
    }
    return hipGetLastError();
}

}  // namespace ctqw
