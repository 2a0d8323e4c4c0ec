// One particle on a general graph (Sec. 2: node a couples to its own set of
// neighbours; a q-dimensional lattice is one such graph), R statically noisy
// realisations sharing one topology, advanced by the truncated Taylor series
// of exp(-i H dt) (Eqs. 5-7) one term per pass: term j is
//     Phi^(j) = (-i dt / j) H Phi^(j-1),   psi(t + dt) = sum_j Phi^(j),
// with H psi gathered through an ELL neighbour table.  The topology is the
// same for every realisation, the couplings and on-site energies are each
// realisation's own.  Complex128 with FP64 tables, or complex64 with FP32
// tables (plain sums); the optional per-step norms are FP64 either way.
//
// Work mapping: one thread per node and group of realisations (four for
// complex64, one for complex128); nodes along the threads (coalesced reads of
// the ELL slots, the couplings, the on-site energies and the state).  Where
// the groups fill the eight XCDs about evenly, a group's blocks all go to one
// XCD: its L2 then fetches that group's previous term once, where blocks
// dealt in turn have every XCD fetch every realisation.  Otherwise the blocks
// run along x and the groups, strided, along y.
// Per node, term and realisation the pass reads the previous term at the
// node and its neighbours, width couplings and slot indices and the on-site
// energy and writes the term.  Only every second term touches the partial sum: the
// term before it is the node's own value of the source, which is at hand, so
// the sum takes both in the order of one after the other (the same bits, 32
// of 136 bytes less in every second term of a complex128 graph of width 8).
// The step's squared norms are block sums of its last term.
// Bound by the couplings' traffic.  Two bosons on 15 x 15 nodes (25425 states,
// width 8), 32 realisations, complex128: 26.3 -> 17.7 us per term (98 MB on
// average: 5.5 TB/s), with every slot's loads behind the previous slot's branch
// before; the step's norms, one block per realisation before, 28.8 -> 5.1 us.
// 24 x 24 nodes, 16 realisations, 127 -> 68 us; one walker on 128 x 128, 256
// realisations, 92 -> 66 (complex64 46 -> 31).
#include "graph.hpp"
#include "wave_sum.hpp"

#include <algorithm>
#include <type_traits>

namespace ctqw {
namespace {

template <typename T> struct Cplx;
template <> struct Cplx<float> { using type = float2; };
template <> struct Cplx<double> { using type = double2; };

__device__ inline float fma_r(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ inline double fma_r(double a, double b, double c) { return __builtin_fma(a, b, c); }

// Realisations per thread: they share the slot indices, and their gathers
// are independent loads in flight together.  Measured on the 128 x 128
// lattice with 4096 realisations: four per thread is 14 % faster for
// complex64 (8-byte gathers) and 19 % slower for complex128, which keeps one.
template <typename T> struct RealsPerThread;
template <> struct RealsPerThread<float> { static constexpr int value = 4; };
template <> struct RealsPerThread<double> { static constexpr int value = 1; };

// Q: realisations per thread.  NORM: the last term of a step; the block's part
// of the squared norms goes to a.parts (summed over each wave, then over the
// four: one barrier, where a tree in LDS takes ten per realisation).
template <typename T, int Q, bool NORM>
__global__ __launch_bounds__(256) void graph_term_kernel(GraphTermArgs a) {
    using C = typename Cplx<T>::type;
    constexpr int S = 4;   // slots whose loads are in flight together
    __shared__ double part[NORM ? 4 : 1][Q];
    const int64_t n = a.n;
    const T* hop = static_cast<const T*>(a.hop);
    const T* onsite = static_cast<const T*>(a.onsite);
    const C* src = static_cast<const C*>(a.src);
    const T cf = static_cast<T>(a.c);
    const int64_t groups = ((int64_t)a.R + Q - 1) / Q;
    int32_t bx = (int32_t)blockIdx.x;
    int64_t g0 = blockIdx.y, step = gridDim.y;
    if (a.by_xcd) {   // one group per block
        const uint32_t k = blockIdx.x >> 3;
        bx = (int32_t)(k % (uint32_t)a.node_blocks);
        g0 = (int64_t)(k / (uint32_t)a.node_blocks) * 8 + (blockIdx.x & 7);
        step = groups;
    }
    const int64_t i = (int64_t)bx * 256 + threadIdx.x;
    const bool in = i < n;
    const int32_t ic = in ? (int32_t)i : 0;   // threads past the end load node 0 and store nothing
    for (int64_t g = g0; g < groups; g += step) {
        const int64_t r0 = g * Q;
        const int nr = (int)((int64_t)a.R - r0 < Q ? (int64_t)a.R - r0 : Q);
        // rows of this group's realisations; a missing one repeats the first
        int64_t row[Q];
        T hr[Q], hi[Q];
        C x[Q];
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            row[q] = r0 + (q < nr ? q : 0);
            x[q] = src[row[q] * n + ic];
            const T e = onsite[row[q] * n + ic];
            hr[q] = e * x[q].x;
            hi[q] = e * x[q].y;
        }
        // No branch around the loads: an empty slot reads node i and its sum
        // is dropped.  One realisation per thread: after a group with empty slots
        // the next is looked at first (its couplings then wait for the indices)
        // and passed over if it is empty at all of the wave's nodes.
        bool gaps = false;
        int32_t k0 = 0;
        auto slots = [&](auto count) {
            constexpr int M = decltype(count)::value;
            constexpr bool LOOK = Q == 1 && M == S;
            int32_t j[M];
            bool has[M], any = false, all = true;
            T c[M][Q];
            C xj[M][Q];
            auto couplings = [&]() {
#pragma unroll
                for (int k = 0; k < M; ++k)
#pragma unroll
                    for (int q = 0; q < Q; ++q) c[k][q] = hop[(row[q] * a.width + k0 + k) * n + ic];
            };
#pragma unroll
            for (int k = 0; k < M; ++k) j[k] = a.nbr[(int64_t)(k0 + k) * n + ic];
            if (!LOOK || !gaps) couplings();
#pragma unroll
            for (int k = 0; k < M; ++k) {
                has[k] = j[k] >= 0 && j[k] < a.n;
                any = any || has[k];
                all = all && has[k];
                j[k] = has[k] ? j[k] : ic;
            }
            if (LOOK && gaps) {
                if (__builtin_amdgcn_ballot_w64(any) == 0) {
                    k0 += M;
                    return;
                }
                couplings();
            }
#pragma unroll
            for (int k = 0; k < M; ++k)
#pragma unroll
                for (int q = 0; q < Q; ++q) xj[k][q] = src[row[q] * n + j[k]];
#pragma unroll
            for (int k = 0; k < M; ++k)
#pragma unroll
                for (int q = 0; q < Q; ++q) {
                    hr[q] = has[k] ? fma_r(c[k][q], xj[k][q].x, hr[q]) : hr[q];
                    hi[q] = has[k] ? fma_r(c[k][q], xj[k][q].y, hi[q]) : hi[q];
                }
            if constexpr (LOOK) gaps = __builtin_amdgcn_ballot_w64(!all) != 0;
            k0 += M;
        };
        while (k0 + S <= a.width) slots(std::integral_constant<int, S>{});
        while (k0 < a.width) slots(std::integral_constant<int, 1>{});
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const bool mine = in && q < nr;
            const int64_t o = row[q] * n + ic;
            // (-i c) (hr + i hi) = c hi - i c hr
            C t;
            t.x = cf * hi[q];
            t.y = -cf * hr[q];
            if (a.t_out && mine) static_cast<C*>(a.t_out)[o] = t;
            double n2 = 0.0;
            if (a.acc_out && mine) {
                C s = static_cast<const C*>(a.acc_in)[o];
                if (a.add_src) {
                    s.x += x[q].x;
                    s.y += x[q].y;
                }
                s.x += t.x;
                s.y += t.y;
                static_cast<C*>(a.acc_out)[o] = s;
                const double re = s.x, im = s.y;
                n2 = fma(re, re, im * im);
            }
            if constexpr (NORM) {
                const double sum = wave_sum_last(n2);
                if ((threadIdx.x & 63) == 63) part[threadIdx.x >> 6][q] = sum;
            }
        }
        if constexpr (NORM) {
            __syncthreads();
            const int q = (int)threadIdx.x;
            if (q < nr) a.parts[(r0 + q) * a.node_blocks + bx] = ((part[0][q] + part[1][q]) + part[2][q]) + part[3][q];
            __syncthreads();
        }
    }
}

// out[r]: the parts of one realisation, in a fixed order.
__global__ __launch_bounds__(256) void graph_norm_kernel(const double* parts, int32_t per_real, double* out) {
    __shared__ double part[4];
    const double* x = parts + blockIdx.x * (int64_t)per_real;
    double acc = 0.0;
    for (int32_t i = (int32_t)threadIdx.x; i < per_real; i += 256) acc += x[i];
    acc = wave_sum_last(acc);
    if ((threadIdx.x & 63) == 63) part[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) out[blockIdx.x] = ((part[0] + part[1]) + part[2]) + part[3];
}

template <typename T, int Q>
hipError_t launch_term(GraphTermArgs a, hipStream_t s) {
    const int64_t groups = ((int64_t)a.R + Q - 1) / Q;
    a.node_blocks = (int32_t)(((int64_t)a.n + 255) / 256);
    // One XCD per group where the fullest XCD has at most a quarter more than
    // an even share.  Per term and step in turn -> by XCD, two bosons on 15 x
    // 15, complex128: R = 8 8.5 -> 7.0 us, 14 (share 1.14) 11.9 -> 11.2, 33
    // (1.21) 23.4 -> 20.5; 12 (1.33) 10.5 -> 11.2, 9 (1.78) 8.9 -> 10.1.
    const int64_t rounds = (groups + 7) / 8, blocks = rounds * 8 * a.node_blocks;
    // (A launch takes fewer than 2^32 threads along x.)
    a.by_xcd = rounds * 8 * 4 <= groups * 5 && blocks < int64_t(1) << 24;
    const dim3 grid = a.by_xcd ? dim3((unsigned)blocks)
                               : dim3((unsigned)a.node_blocks, (unsigned)std::min<int64_t>(groups, 65535));
    if (a.parts) hipLaunchKernelGGL((graph_term_kernel<T, Q, true>), grid, dim3(256), 0, s, a);
    else hipLaunchKernelGGL((graph_term_kernel<T, Q, false>), grid, dim3(256), 0, s, a);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_graph_term(const GraphTermArgs& a, int dtype, hipStream_t s) {
    if (dtype == 1) return launch_term<double, RealsPerThread<double>::value>(a, s);
    // fewer realisations than a thread's share would repeat one of them (one
    // realisation of 5000 nodes, width 12, 3 steps of 8 terms: 228 us in fours, 141)
    constexpr int Q = RealsPerThread<float>::value;
    return a.R < Q ? launch_term<float, 1>(a, s) : launch_term<float, Q>(a, s);
}

hipError_t launch_graph_norms(const double* parts, int32_t n, int32_t R, double* out, hipStream_t s) {
    hipLaunchKernelGGL(graph_norm_kernel, dim3((unsigned)R), dim3(256), 0, s, parts, (int32_t)(((int64_t)n + 255) / 256),
                       out);
    return hipGetLastError();
}

}  // namespace ctqw
