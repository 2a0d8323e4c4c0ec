// Hermitian rank-R update of the ensemble-averaged density matrix (Eq. 2),
//     rho = (1/R) sum_r |a_r><a_r| = A A^H / R,   A: D x R complex,
// on the matrix cores, lower triangle only.  The paper forms rho with one
// rank-1 update per realisation; here the R rank-1 updates are one
// contraction over r.
//
// With a = ar + i ai, a product term a_i conj(a_j) is
//     Re = ar_i ar_j + ai_i ai_j,      Im = ai_i ar_j - ar_i ai_j,
// i.e. two real inner products of length 2 per realisation: the real and
// imaginary parts of one complex entry are the two k-slots of one MFMA
// step.  For complex64, v_mfma_f32_32x32x2_f32 takes, per lane l, the
// A entry of row l % 32 and k-slot l / 32, and the B entry of the same
// k-slot and column l % 32: with A = (ar_i, ai_i) and B = (ar_j, ai_j) it
// accumulates Re; with A' = (ai_i, -ar_i) and the same B, Im.  For
// complex128, v_mfma_f64_16x16x4_f64 takes four k-slots: two complex
// realisations per step.
//
// Input: the group's gathered states in split planes [re / im][Rp][Dp]
// (realisation-major, each realisation's D entries contiguous, zero padding
// up to Dp rows and Rp realisations), so that every tile and stage is
// loaded without bounds tests.  Work item: one tile of the lower triangle.
// The product is formed for the transposed tile -- MFMA rows from the
// tile's column block, MFMA columns from its row block -- so that each
// lane's accumulators hold consecutive rows of rho in column-major order
// and the conjugated values are stored 256 contiguous bytes per half-wave.
// Tiles on the diagonal store only their lower part; diagonal entries are
// stored with imaginary part 0 (rho is Hermitian).
#include "density.hpp"

namespace ctqw {
namespace herk_detail {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef double doublex4 __attribute__((ext_vector_type(4)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

// Tile index t -> (P, Q), P >= Q, row-major over the lower triangle.
__device__ __forceinline__ void tile_of(int64_t t, int* P, int* Q) {
    int p = (int)((sqrt(8.0 * (double)t + 1.0) - 1.0) * 0.5);
    while ((int64_t)(p + 1) * (p + 2) / 2 <= t) ++p;
    while ((int64_t)p * (p + 1) / 2 > t) --p;
    *P = p;
    *Q = (int)(t - (int64_t)p * (p + 1) / 2);
}

// The tile of this block.  NB = 2: tile a.tile0 + k, k dealt to the XCDs in
// consecutive runs.  NB = 1: a quarter of one, tiles of half the side (none
// above the diagonal).  Returns false for blocks without a tile.
template <int NB>
__device__ __forceinline__ bool my_tile(const HerkArgs& a, int* P, int* Q) {
    if constexpr (NB == 2) {
        const int per_xcd = (int)((a.n_tiles + 7) / 8);
        const int64_t t = (int64_t)(blockIdx.x % 8) * per_xcd + (blockIdx.x / 8);
        if (t >= a.n_tiles) return false;
        tile_of(a.tile0 + t, P, Q);
    } else {
        tile_of(a.tile0 + blockIdx.x / 4, P, Q);
        *P = 2 * *P + (int)(blockIdx.x & 1);
        *Q = 2 * *Q + (int)((blockIdx.x >> 1) & 1);
        if (*P < *Q) return false;
    }
    return true;
}

// complex64: block tile 64 NB square, 4 waves of NB x NB MFMA blocks of
// 32 x 32, stages of KC = 16 realisations staged in LDS, double-buffered.
constexpr int TS = 128;
constexpr int KC = 16;

template <int NB>
__global__ void __launch_bounds__(256, 2) herk_c64_kernel(HerkArgs a) {
    constexpr int TS = 64 * NB;
    __shared__ float lds[2][2][2][KC][TS];   // [buffer][panel: col block Q, row block P][plane][k][row]
    int P, Q;
    if (!my_tile<NB>(a, &P, &Q)) return;   // whole block, before any barrier
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int w = tid >> 6;
    const int wr = w >> 1, wc = w & 1;          // wave's sub-tile: MFMA rows (Q side), columns (P side)
    const int64_t Dp = a.Dp, plane = (int64_t)a.Rp * Dp;
    const float* G = static_cast<const float*>(a.G);
    const int64_t q0 = (int64_t)Q * TS, p0 = (int64_t)P * TS;

    // stage loads: 2 panels x 2 planes x KC x TS floats = 1024 NB float4, 4 NB per thread
    floatx4 st[4 * NB];
    constexpr int Q4 = TS / 4;                  // float4 of one row of a stage
    auto load_stage = [&](int k0) {
#pragma unroll
        for (int u = 0; u < 4 * NB; ++u) {
            const int f = tid + 256 * u;            // [panel][plane][k][row4]
            const int panel = f / (2 * KC * Q4), pl = (f / (KC * Q4)) & 1, kk = (f / Q4) % KC, r4 = f % Q4;
            const int64_t base = (panel == 0 ? q0 : p0) + 4 * r4;
            st[u] = *reinterpret_cast<const floatx4*>(G + pl * plane + (int64_t)(k0 + kk) * Dp + base);
        }
    };
    auto store_stage = [&](int b) {
#pragma unroll
        for (int u = 0; u < 4 * NB; ++u) {
            const int f = tid + 256 * u;
            const int panel = f / (2 * KC * Q4), pl = (f / (KC * Q4)) & 1, kk = (f / Q4) % KC, r4 = f % Q4;
            *reinterpret_cast<floatx4*>(&lds[b][panel][pl][kk][4 * r4]) = st[u];
        }
    };

    floatx16 accR[NB][NB], accI[NB][NB];
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) accR[i][j][e] = accI[i][j][e] = 0.0f;

    const int kslot = lane >> 5;          // 0: real part, 1: imaginary part
    const int row = lane & 31;
    const float sgn = kslot ? -1.0f : 1.0f;
    const int stages = a.Rp / KC;
    load_stage(0);
    store_stage(0);
    __syncthreads();
    for (int s = 0; s < stages; ++s) {
        const int b = s & 1;
        if (s + 1 < stages) load_stage((s + 1) * KC);
#pragma unroll 4
        for (int kk = 0; kk < KC; ++kk) {
            float av[NB], ap[NB], bv[NB];
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                const int m = 32 * NB * wr + 32 * i + row;
                av[i] = lds[b][0][kslot][kk][m];
                ap[i] = sgn * lds[b][0][1 - kslot][kk][m];
                const int n = 32 * NB * wc + 32 * i + row;
                bv[i] = lds[b][1][kslot][kk][n];
            }
#pragma unroll
            for (int i = 0; i < NB; ++i)
#pragma unroll
                for (int j = 0; j < NB; ++j) {
                    accR[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(av[i], bv[j], accR[i][j], 0, 0, 0);
                    accI[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(ap[i], bv[j], accI[i][j], 0, 0, 0);
                }
        }
        if (s + 1 < stages) {
            store_stage(b ^ 1);
            __syncthreads();
        }
    }

    // C'[m][n] = sum a_{Q,m} conj(a_{P,n}) = rho[Q m][P n]; rho[P n][Q m] = conj(C'[m][n]).
    // Accumulator e of a lane: MFMA row m = 8 (e / 4) + 4 (lane / 32) + e % 4, column n = lane % 32.
    const float inv = (float)a.inv_R;
    float2* rho = static_cast<float2*>(a.rho);
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int m = 8 * (e >> 2) + 4 * kslot + (e & 3);
                const int64_t gc = q0 + 32 * NB * wr + 32 * i + m;     // rho column
                const int64_t gr = p0 + 32 * NB * wc + 32 * j + row;   // rho row
                if (gr < a.D && gc < a.D && (P != Q || gr >= gc)) {
                    float2 v;
                    v.x = accR[i][j][e] * inv;
                    v.y = gr == gc ? 0.0f : -accI[i][j][e] * inv;   // Hermitian: real diagonal
                    rho[gr + (int64_t)a.ld * gc] = v;
                }
            }
}

// complex128: block tile 32 NB square, 4 waves of NB x NB MFMA blocks of
// 16 x 16, v_mfma_f64_16x16x4_f64 with k-slots (re, im) of two
// realisations per step; stages of 8 realisations.
constexpr int TS2 = 64;
constexpr int KC2 = 8;

template <int NB>
__global__ void __launch_bounds__(256, 2) herk_c128_kernel(HerkArgs a) {
    constexpr int TS2 = 32 * NB;
    __shared__ double lds[2][2][2][KC2][TS2];   // [buffer][panel][plane][k][row]
    int P, Q;
    if (!my_tile<NB>(a, &P, &Q)) return;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int w = tid >> 6;
    const int wr = w >> 1, wc = w & 1;
    const int64_t Dp = a.Dp, plane = (int64_t)a.Rp * Dp;
    const double* G = static_cast<const double*>(a.G);
    const int64_t q0 = (int64_t)Q * TS2, p0 = (int64_t)P * TS2;

    // stage: 2 panels x 2 planes x 8 x TS2 doubles = 512 NB double2, 2 NB per thread
    typedef double doublex2 __attribute__((ext_vector_type(2)));
    doublex2 st[2 * NB];
    constexpr int Q2 = TS2 / 2;                 // double2 of one row of a stage
    auto load_stage = [&](int k0) {
#pragma unroll
        for (int u = 0; u < 2 * NB; ++u) {
            const int f = tid + 256 * u;            // [panel][plane][k][row2]
            const int panel = f / (2 * KC2 * Q2), pl = (f / (KC2 * Q2)) & 1, kk = (f / Q2) % KC2, r2 = f % Q2;
            const int64_t base = (panel == 0 ? q0 : p0) + 2 * r2;
            st[u] = *reinterpret_cast<const doublex2*>(G + pl * plane + (int64_t)(k0 + kk) * Dp + base);
        }
    };
    auto store_stage = [&](int b) {
#pragma unroll
        for (int u = 0; u < 2 * NB; ++u) {
            const int f = tid + 256 * u;
            const int panel = f / (2 * KC2 * Q2), pl = (f / (KC2 * Q2)) & 1, kk = (f / Q2) % KC2, r2 = f % Q2;
            *reinterpret_cast<doublex2*>(&lds[b][panel][pl][kk][2 * r2]) = st[u];
        }
    };

    doublex4 accR[NB][NB], accI[NB][NB];
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) accR[i][j][e] = accI[i][j][e] = 0.0;

    const int kslot = lane >> 4;          // 0..3: realisation kk + (kslot >> 1), part kslot & 1
    const int part = kslot & 1, sub = kslot >> 1;
    const int row = lane & 15;
    const double sgn = part ? -1.0 : 1.0;
    const int stages = a.Rp / KC2;
    load_stage(0);
    store_stage(0);
    __syncthreads();
    for (int s = 0; s < stages; ++s) {
        const int b = s & 1;
        if (s + 1 < stages) load_stage((s + 1) * KC2);
#pragma unroll
        for (int kk = 0; kk < KC2; kk += 2) {
            double av[NB], ap[NB], bv[NB];
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                const int m = 16 * NB * wr + 16 * i + row;
                av[i] = lds[b][0][part][kk + sub][m];
                ap[i] = sgn * lds[b][0][1 - part][kk + sub][m];
                const int n = 16 * NB * wc + 16 * i + row;
                bv[i] = lds[b][1][part][kk + sub][n];
            }
#pragma unroll
            for (int i = 0; i < NB; ++i)
#pragma unroll
                for (int j = 0; j < NB; ++j) {
                    accR[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[i], bv[j], accR[i][j], 0, 0, 0);
                    accI[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(ap[i], bv[j], accI[i][j], 0, 0, 0);
                }
        }
        if (s + 1 < stages) {
            store_stage(b ^ 1);
            __syncthreads();
        }
    }

    // accumulator e of a lane: MFMA row m = 4 e + lane / 16, column n = lane % 16
    const double inv = a.inv_R;
    double2* rho = static_cast<double2*>(a.rho);
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int m = 4 * e + kslot;
                const int64_t gc = q0 + 16 * NB * wr + 16 * i + m;
                const int64_t gr = p0 + 16 * NB * wc + 16 * j + row;
                if (gr < a.D && gc < a.D && (P != Q || gr >= gc)) {
                    double2 v;
                    v.x = accR[i][j][e] * inv;
                    v.y = gr == gc ? 0.0 : -accI[i][j][e] * inv;    // Hermitian: real diagonal
                    rho[gr + (int64_t)a.ld * gc] = v;
                }
            }
}

}  // namespace herk_detail

int herk_tile(int dtype) { return dtype == 1 ? herk_detail::TS2 : herk_detail::TS; }
int herk_stage(int dtype) { return dtype == 1 ? herk_detail::KC2 : herk_detail::KC; }

// Bound by the matrix cores: the whole tiles keep them 84.5 % busy (2.33 GHz).
// Two blocks of a whole tile fit a compute unit, 512 the device, and they all
// take the same time, so whole tiles go in full rounds of 512.  The tiles
// past the last full round go in quarters while those still take less than a
// round: four times the blocks, each with a quarter of the products and half
// the operands.  Measured, round of whole tiles -> quarters, complex64:
// two bosons, R = 1000, N = 128 (2145 tiles, 97 past four rounds) 2.46 ->
// 2.34 ms, N = 64 (153 tiles) 0.344 -> 0.267, N = 32 (15 tiles) 0.323 ->
// 0.127; R = 500, N = 101 (349 past a round) 0.621 -> 0.574.  complex128:
// R = 1000, N = 32 0.203 -> 0.106 ms.  After whole rounds that is a second launch,
// 3 us, which few realisations do not win back (us of a call, all whole -> with
// quarters: complex128 N = 66, 118 tiles past a round, R = 24 59.6 -> 63.7, 128
// 96.1 -> 96.2, 256 145.6 -> 142.8; complex64 N = 101 R = 16 101.0 -> 104.6, 24
// 117.2 -> 116.8).
hipError_t launch_herk(const HerkArgs& a, int dtype, hipStream_t s) {
    if (a.n_tiles <= 0) return hipSuccess;
    constexpr int64_t kRound = 512, kQuarters = 384;
    int64_t tail = a.n_tiles % kRound;
    if (tail > kQuarters || (a.n_tiles > kRound && a.Rp < (dtype == 1 ? 128 : 32))) tail = 0;
    HerkArgs whole = a, quarter = a;
    whole.tile0 = 0;
    whole.n_tiles = a.n_tiles - tail;
    quarter.tile0 = whole.n_tiles;
    quarter.n_tiles = tail;
    const int64_t blocks = ((whole.n_tiles + 7) / 8) * 8;
    if (blocks > INT32_MAX) return hipErrorInvalidValue;
    using namespace herk_detail;
    if (dtype == 1) {
        if (blocks) hipLaunchKernelGGL(herk_c128_kernel<2>, dim3((unsigned)blocks), dim3(256), 0, s, whole);
        if (tail) hipLaunchKernelGGL(herk_c128_kernel<1>, dim3((unsigned)(4 * tail)), dim3(256), 0, s, quarter);
    } else {
        if (blocks) hipLaunchKernelGGL(herk_c64_kernel<2>, dim3((unsigned)blocks), dim3(256), 0, s, whole);
        if (tail) hipLaunchKernelGGL(herk_c64_kernel<1>, dim3((unsigned)(4 * tail)), dim3(256), 0, s, quarter);
    }
    return hipGetLastError();
}

}  // namespace ctqw
