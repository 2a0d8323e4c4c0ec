// Two walkers on a small lattice: whole runs of steps with the state on chip.
//
// One block owns one realisation and holds its state in registers from the
// first step of the launch to the last; HBM sees one read and one write of
// the state per launch instead of per step, and a launch replaces two per
// step (the step kernel and its norm check).  The terms of Alg. 3 (Eqs. 6-7)
// are formed level by level in place: a wave holds S consecutive rows, 64 P
// columns wide, so a neighbour is a register (rows), a DPP lane shift
// (columns) or, at the edges of a wave's rows, a row published in LDS by the
// wave next to it -- one barrier per level, nothing recomputed.
//
// What bounds it: the vector ALUs' issue, 32 instructions per row of 128
// complex128 amplitudes and level (24 products and sums, 8 lane shifts), and
// what the waves of a block cannot hide of the exchange at each level.  1000
// realisations of two bosons on 128 nodes, complex128, 12 terms: 90 us per
// step (733 with swept bands and a pass over the state per step), the SIMDs'
// VALUs about 65 % busy at the 2.1 GHz such runs hold; 132 MB of states are
// read and written once per launch, so HBM is idle.
//
// Rows and columns of the held grid:
//  * full grid (open or ring): row k = x1, column p = x2;
//  * triangle (two bosons or fermions, the symmetric or antisymmetric function
//    stored on x1 <= x2): by cyclic difference, row k = 0 .. N/2, column
//    p = 0 .. N-1 holds the pair {p, q}, q = (p + k) mod N.  The rows are all
//    full (N(N/2 + 1) slots for N(N+1)/2 amplitudes, where the square would
//    take N^2), a move of p or q changes k by one at column p or p +- 1, and
//    the chain's missing bond N-1 (coupling 0) separates the pairs that wrap.
//    Row -1 is row 1 shifted by one column (a pair's two orders), which also
//    gives the doubled couplings of a doubly occupied node; row N/2 + 1 is
//    the row of difference N - (N/2 + 1), rotated.  For even N the pairs of
//    row N/2 are held twice and weigh half.
// A row past the grid has zero couplings and stays zero, except that the
// slot after the grid's last row carries that row's neighbour.
#pragma once

#include "resident.hpp"
#include "step2d_impl.hpp"
#include "wave_sum.hpp"

namespace ctqw {
namespace resident_detail {

using step2d_detail::CplxOf;
using step2d_detail::UniformPtr;
using step2d_detail::fma_t;
using step2d_detail::from_left;
using step2d_detail::from_right;
using step2d_detail::load_uniform;

// Storage index of {x1, x2}, x1 <= x2, in the triangle.
__device__ __forceinline__ int tri_at(int a, int b, int N) { return a * N - (a * (a + 1)) / 2 + b; }

// The same value, opaque to the optimiser: comparisons of it are made where
// they are needed instead of once before the run (a mask of two scalar
// registers for each row slot, which would spill).
__device__ __forceinline__ int here(int x) {
    asm volatile("" : "+s"(x));
    return x;
}

template <typename T>
__device__ __forceinline__ T lane_value(T x, int lane);
template <>
__device__ __forceinline__ float lane_value<float>(float x, int lane) {
    return __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(x), lane));
}
template <>
__device__ __forceinline__ double lane_value<double>(double x, int lane) {
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x), lane),
                            __builtin_amdgcn_readlane(__double2loint(x), lane));
}

// Calls f(0), f(1), .. f(N - 1) with compile-time slots.
template <int N, int I = 0, typename F>
__device__ __forceinline__ void each_slot(F f) {
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        each_slot<N, I + 1>(f);
    }
}
// Marks a branch that differs from others only in its row slot, so that they
// are not merged into one with a computed slot (which would move the row
// arrays out of registers).
template <int S>
__device__ __forceinline__ void own_branch() {
    asm volatile("; slot %0" ::"n"(S));
}

// LDS of one block: two sets of published rows, the diagonal of dt H on the
// held grid (rows of diag_stride(N) entries), TRI: the bonds, and the norm
// partials.
template <int P>
__host__ __device__ constexpr int diag_stride(int N) { return P == 1 ? N : (N + 1) & ~1; }
// Bonds J[x mod N], x = -1 .. 64 P + rows, even and odd x apart (so that the
// lanes of a wave, P entries apart, read neighbouring words).
template <int P>
__host__ __device__ constexpr int bond_plane() { return 64 + 80; }

template <typename T, int LAYOUT, int P, int S, bool KAHAN, int MAXT>
__global__ void __launch_bounds__(MAXT) resident_kernel(ResidentArgs a) {
    using C = typename CplxOf<T>::type;
    constexpr bool TRI = LAYOUT == kResTri;
    constexpr bool RING = LAYOUT == kResRing;
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int W = blockDim.x >> 6;
    const int r = blockIdx.x;
    const RealDev rd = load_uniform(a.reals, r);
    const int N = rd.N;
    const int K = TRI ? N / 2 + 1 : N;            // rows of the held grid
    const int k0 = wv * S;
    const int kx = TRI ? N - K : K - 1;           // the extra published row
    const int top = K - 1 - k0;                   // this wave's slot of the last row (if 0 <= top < S)
    const bool fermi = TRI && (rd.flags & RF_FERMION) != 0;
    const bool nearest = (rd.flags & RF_NEAREST) != 0;
    const T Udt = static_cast<T>(rd.U * a.dt);
    const UniformPtr<T> Ju_tab = (UniformPtr<T>)((const T*)a.Jt + rd.param_off);
    const T* __restrict__ Jg = (const T*)a.Jt + rd.param_off;
    const T* __restrict__ Eg = (const T*)a.Et + rd.param_off;
    const C* psi = reinterpret_cast<const C*>(a.psi_in) + rd.state_off;

    extern __shared__ char lds_raw[];
    // Published rows: [2][2 W + 3][64 P] -- first and last row of every wave,
    // row kx, TRI: row 1, and a row of zeros.
    C* pub = reinterpret_cast<C*>(lds_raw);
    const int slots = 2 * W + 3;
    const int slot_x = 2 * W, slot_1 = 2 * W + 1, slot_z = 2 * W + 2;
    for (int i = threadIdx.x; i < 2 * 64 * P; i += blockDim.x) {
        C z;
        z.x = z.y = T(0);
        pub[((i / (64 * P)) * slots + slot_z) * 64 * P + i % (64 * P)] = z;
    }
    double* part = reinterpret_cast<double*>(pub + 2 * slots * 64 * P);   // [2][W][2]
    T* tabJ = reinterpret_cast<T*>(part + 4 * W);                         // TRI: [P][bond_plane]
    T* tabD = tabJ + (TRI ? P * bond_plane<P>() : 0);                     // [K][diag_stride]
    const int ds = diag_stride<P>(N);

    if constexpr (TRI) {
        for (int i = threadIdx.x; i < P * bond_plane<P>(); i += blockDim.x) {
            const int plane = i / bond_plane<P>(), at = i % bond_plane<P>();
            tabJ[i] = Jg[(at * P + plane + N - 1) % N];   // entry e is J[e - 1]
        }
    }
    for (int i = threadIdx.x; i < K * ds; i += blockDim.x) {
        const int k = i / ds, c = i % ds;
        T d = T(0);
        if (c < N) {
            int q = TRI ? c + k : k;
            if (TRI && q >= N) q -= N;
            const int x = abs(q - c);   // chain distance of the pair
            const bool hit = nearest ? (x == 1 || (RING && x == N - 1)) : x == 0;
            d = Eg[c] + Eg[q] + (hit ? Udt : T(0));
        }
        tabD[i] = d;
    }

    int col[P];
    bool in[P];
    T jl[P], jr[P];
#pragma unroll
    for (int p = 0; p < P; ++p) {
        col[p] = lane * P + p;
        in[p] = col[p] < N;
        const int c = in[p] ? col[p] : 0;
        jl[p] = in[p] ? Jg[c == 0 ? N - 1 : c - 1] : T(0);
        jr[p] = in[p] ? Jg[c] : T(0);
    }

    // Row tables of the full grid (wave-uniform); rows past the grid: 0.
    T ju[S + 1];
    if constexpr (!TRI) {
#pragma unroll
        for (int s = 0; s < S; ++s) {
            const int k = k0 + s;
            // (the slot after the last row holds the bond below that row)
            ju[s] = (k < K || (k == K && s > 0)) ? Ju_tab[k == 0 ? N - 1 : k - 1] : T(0);
        }
        {
            const int k = k0 + S - 1;
            ju[S] = k < K ? Ju_tab[k] : T(0);
        }
    }

    // Stored element of (slot s, column c), or -1.
    auto element = [&](int kb, int s, int c) -> int {
        const int k = kb + s;
        if (k >= K || c >= N) return -1;
        if constexpr (TRI) {
            int q = c + k;
            if (q >= N) q -= N;
            return tri_at(min(c, q), max(c, q), N);
        } else {
            return k * N + c;
        }
    };

    T tr[S][P], ti[S][P];           // the level's vector, Y_j = (dt H)^j psi
    T ar[S][P], ai[S][P];           // sum of the terms (KAHAN: of j >= 1)
    T pr[KAHAN ? S : 1][P], pi[KAHAN ? S : 1][P];   // KAHAN: the state
    double sc = ((UniformPtr<double>)a.scale)[r];
#pragma unroll
    for (int s = 0; s < S; ++s)
#pragma unroll
        for (int p = 0; p < P; ++p) {
            const int e = element(k0, s, col[p]);
            tr[s][p] = ti[s][p] = T(0);
            if (e >= 0) {
                const C v = psi[e];
                tr[s][p] = v.x;
                ti[s][p] = v.y;
            }
        }

    const int n = a.one_order > 0 ? a.one_order : rd.order;
    const double tf = a.one_order > 0 ? rd.tail_factor_max : rd.tail_factor;

    // Publish row slot s of the vector for the neighbouring waves (columns of
    // one lane 64 elements apart: no bank conflicts).
    auto put = [&](C* dst, auto s) {
        C v[P];
#pragma unroll
        for (int p = 0; p < P; ++p) {
            v[p].x = tr[s][p];
            v[p].y = ti[s][p];
        }
        own_branch<s>();
#pragma unroll
        for (int p = 0; p < P; ++p) dst[p * 64 + lane] = v[p];
    };
    auto publish = [&](int b) {
        C* base = pub + b * slots * 64 * P;
        put(base + (2 * wv) * 64 * P, std::integral_constant<int, 0>{});
        put(base + (2 * wv + 1) * 64 * P, std::integral_constant<int, S - 1>{});
        if constexpr (LAYOUT != kResFull) {
            if (kx >= k0 && kx < k0 + S) {
                const int x = here(kx - k0);
                each_slot<S>([&](auto s) {
                    if (x == s) put(base + slot_x * 64 * P, s);
                });
            }
        }
        if constexpr (TRI) {
            if (k0 == 0) put(base + slot_1 * 64 * P, std::integral_constant<int, 1>{});
        }
    };

    int buf = 0;
    // The rows above the wave's first and below its last, as elements of the
    // published rows (the row of zeros off an open grid and off the chain).
    const bool is_top = top >= 0 && top < S;
    const bool early_top = LAYOUT != kResFull && is_top && top < S - 1;
    const int lo_slot = k0 > 0 ? 2 * wv - 1 : (RING ? slot_x : slot_z);
    const int hi_slot = top >= S ? 2 * wv + 2 : (is_top && LAYOUT != kResFull ? (RING ? 0 : slot_x) : slot_z);
    int lo_at[P], hi_at[P];
#pragma unroll
    for (int p = 0; p < P; ++p) {
        auto element_at = [&](int slot, int c) { return slot * 64 * P + (c % P) * 64 + c / P; };
        const int c = lane * P + p;
        lo_at[p] = element_at(lo_slot, c);
        hi_at[p] = element_at(hi_slot, c);
        if constexpr (TRI) {
            // row -1: row 1 shifted by one column; row N/2 + 1: rotated
            if (k0 == 0) lo_at[p] = c > 0 && in[p] ? element_at(slot_1, c - 1) : element_at(slot_z, c);
            if (is_top) hi_at[p] = in[p] ? element_at(slot_x, c + K >= N ? c + K - N : c + K) : element_at(slot_z, c);
        }
    }
    // This lane's table entries.  Columns off the chain read the first column's
    // diagonal (they hold zeros).
    const T* const dg = tabD + min(k0, K - 1) * ds + (in[0] ? lane * P : 0);
    const int dlast = max(0, K - 1 - k0);
    const T* const bj0 = TRI ? tabJ + (P == 1 ? lane + k0 : (k0 & 1) * bond_plane<P>() + lane + (k0 >> 1)) : nullptr;
    const T* const bj1 = TRI && P == 2 ? tabJ + ((k0 + 1) & 1) * bond_plane<P>() + lane + ((k0 + 1) >> 1) : nullptr;
    // The last level's squares, before the 1/n! that scales them: a triangle's in
    // FP64, as deep series leave FP32's range; a grid's per lane in the state's
    // precision (either as the bands do; FP64 costs the grids 5 %).
    using Tail = std::conditional_t<TRI, double, T>;
    // One level, in place: t <- (dt H) t; the sum takes the new vector with
    // the factor (-i)^j / j!: ODD levels swap the parts.  Rows 1 .. S - 1
    // first, then row 0: the neighbouring waves' rows are needed last.
    auto level = [&](auto odd, T c, bool last, Tail& tail) {
        constexpr bool ODD = decltype(odd)::value;
        const C* base = pub + buf * slots * 64 * P;
        T lr[P], li[P], hr[P], hi[P];
        auto read_hi = [&]() {
#pragma unroll
            for (int p = 0; p < P; ++p) {
                const C v = base[hi_at[p]];
                hr[p] = v.x;
                hi[p] = v.y;
            }
        };
        auto read_lo = [&]() {
#pragma unroll
            for (int p = 0; p < P; ++p) {
                const C v = base[lo_at[p]];
                lr[p] = v.x;
                li[p] = v.y;
            }
        };
        if (early_top) {            // the row after the grid's last, in its slot
            read_hi();
            const int t = here(top);
            each_slot<S - 1>([&](auto s) {
                if (t == s) {
#pragma unroll
                    for (int p = 0; p < P; ++p) { tr[s + 1][p] = hr[p]; ti[s + 1][p] = hi[p]; }
                    own_branch<s>();
                }
            });
        }
        // Table entries, read AHEAD rows before their use: the diagonal (a row past
        // the grid reads the last row's; its values are never used), and for the
        // triangle J[q - 1] .. J[q + P - 1], which slide by one entry per row.
        constexpr int AHEAD = 2;
        T o1r[P], o1i[P];           // row 1, old values
        T ur[P], ui[P];             // the row above, old values
        T wj[TRI ? S + P : 1], dd[S][P];
        auto bond = [&](int i) {
            if constexpr (TRI) wj[i] = P == 1 || i % 2 == 0 ? bj0[i / P] : bj1[i / P];
        };
        auto ahead = [&](int i) {   // what row i needs beyond the rows before it
            if constexpr (TRI) bond(i + P);
            const T* __restrict__ d = dg + min(i, dlast) * ds;
#pragma unroll
            for (int p = 0; p < P; ++p) dd[i][p] = d[p];
        };
        auto row = [&](auto slot, const T (&ur)[P], const T (&ui)[P], const T (&vr)[P], const T (&vi)[P]) {
            constexpr int s = decltype(slot)::value;
            T nr[P], ni[P];
            if constexpr (TRI) {
                // t(k - 1, p + 1) and t(k + 1, p - 1)
                T xr[P], xi[P], yr[P], yi[P];
                xr[P - 1] = from_right(ur[0]);
                xi[P - 1] = from_right(ui[0]);
                yr[0] = from_left(vr[P - 1]);
                yi[0] = from_left(vi[P - 1]);
#pragma unroll
                for (int p = 0; p + 1 < P; ++p) {
                    xr[p] = ur[p + 1];
                    xi[p] = ui[p + 1];
                    yr[p + 1] = vr[p];
                    yi[p + 1] = vi[p];
                }
#pragma unroll
                for (int p = 0; p < P; ++p) {
                    const T jq0 = wj[s + p], jq1 = wj[s + p + 1];   // J[q - 1], J[q]
                    const T d = dd[s][p];
                    T h = d * tr[s][p], g = d * ti[s][p];
                    h = fma_t(jq0, ur[p], h);
                    g = fma_t(jq0, ui[p], g);
                    h = fma_t(jq1, vr[p], h);
                    g = fma_t(jq1, vi[p], g);
                    h = fma_t(jl[p], yr[p], h);
                    g = fma_t(jl[p], yi[p], g);
                    h = fma_t(jr[p], xr[p], h);
                    g = fma_t(jr[p], xi[p], g);
                    if (s == 0 && fermi && k0 == 0) { h = T(0); g = T(0); }
                    nr[p] = h;
                    ni[p] = g;
                }
            } else {
                T xr[P], xi[P], yr[P], yi[P];   // columns p - 1 and p + 1
                xr[0] = from_left(tr[s][P - 1]);
                xi[0] = from_left(ti[s][P - 1]);
                yr[P - 1] = from_right(tr[s][0]);
                yi[P - 1] = from_right(ti[s][0]);
#pragma unroll
                for (int p = 0; p + 1 < P; ++p) {
                    xr[p + 1] = tr[s][p];
                    xi[p + 1] = ti[s][p];
                    yr[p] = tr[s][p + 1];
                    yi[p] = ti[s][p + 1];
                }
                if constexpr (RING) {
                    const int ll = (N - 1) / P;
                    const bool odd_end = P > 1 && (N - 1) % P != 0;
                    const T zr = lane_value(odd_end ? tr[s][P - 1] : tr[s][0], ll);
                    const T zi = lane_value(odd_end ? ti[s][P - 1] : ti[s][0], ll);
                    const T fr = lane_value(tr[s][0], 0), fi = lane_value(ti[s][0], 0);
                    if (lane == 0) { xr[0] = zr; xi[0] = zi; }
#pragma unroll
                    for (int p = 0; p < P; ++p)
                        if (col[p] == N - 1) { yr[p] = fr; yi[p] = fi; }
                }
#pragma unroll
                for (int p = 0; p < P; ++p) {
                    const T d = dd[s][p];
                    T h = d * tr[s][p], g = d * ti[s][p];
                    h = fma_t(ju[s], ur[p], h);
                    g = fma_t(ju[s], ui[p], g);
                    h = fma_t(ju[s + 1], vr[p], h);
                    g = fma_t(ju[s + 1], vi[p], g);
                    h = fma_t(jl[p], xr[p], h);
                    g = fma_t(jl[p], xi[p], g);
                    h = fma_t(jr[p], yr[p], h);
                    g = fma_t(jr[p], yi[p], g);
                    nr[p] = h;
                    ni[p] = g;
                }
            }
#pragma unroll
            for (int p = 0; p < P; ++p) {
                tr[s][p] = nr[p];
                ti[s][p] = ni[p];
                if constexpr (ODD) {
                    ar[s][p] = fma_t(c, ni[p], ar[s][p]);
                    ai[s][p] = fma_t(-c, nr[p], ai[s][p]);
                } else {
                    ar[s][p] = fma_t(c, nr[p], ar[s][p]);
                    ai[s][p] = fma_t(c, ni[p], ai[s][p]);
                }
            }
            // One row's operands at a time: without these the rows' table reads
            // are all brought forward, the sums put off past the barrier, and
            // the vectors spill.
#pragma unroll
            for (int p = 0; p < P; ++p) {
                asm volatile("" : "+v"(tr[s][p]), "+v"(ti[s][p]));
                asm volatile("" : "+v"(ar[s][p]), "+v"(ai[s][p]));
            }
            __builtin_amdgcn_sched_barrier(0);
        };
#pragma unroll
        for (int i = 0; TRI && i < P; ++i) bond(i);
#pragma unroll
        for (int i = 0; i < AHEAD + 1 && i < S; ++i) ahead(i);
#pragma unroll
        for (int p = 0; p < P; ++p) {
            o1r[p] = tr[S > 1 ? 1 : 0][p];
            o1i[p] = ti[S > 1 ? 1 : 0][p];
            ur[p] = tr[0][p];
            ui[p] = ti[0][p];
        }
        if (S <= 3) { read_hi(); read_lo(); }
        each_slot<S - 1>([&](auto before) {
            constexpr int s = decltype(before)::value + 1;
            if (s + AHEAD < S) ahead(s + AHEAD);
            if (S > 3 && s == S - 3) read_hi();
            if (S > 3 && s == S - 2) read_lo();
            T tmr[P], tmi[P], vr[P], vi[P];
#pragma unroll
            for (int p = 0; p < P; ++p) {
                tmr[p] = tr[s][p];
                tmi[p] = ti[s][p];
                vr[p] = s + 1 < S ? tr[s + 1 < S ? s + 1 : s][p] : hr[p];
                vi[p] = s + 1 < S ? ti[s + 1 < S ? s + 1 : s][p] : hi[p];
            }
            row(std::integral_constant<int, s>{}, ur, ui, vr, vi);
#pragma unroll
            for (int p = 0; p < P; ++p) { ur[p] = tmr[p]; ui[p] = tmi[p]; }
        });
        if constexpr (S > 1) row(std::integral_constant<int, 0>{}, lr, li, o1r, o1i);
        else row(std::integral_constant<int, 0>{}, lr, li, hr, hi);
        if (!last) {
            publish(buf ^ 1);
            __syncthreads();
            buf ^= 1;
        } else {
            const int kb = here(k0);
#pragma unroll
            for (int s = 0; s < S; ++s) {
                const int k = kb + s;
                const Tail w = TRI && k != 0 && 2 * k != N ? Tail(2) : Tail(1);
#pragma unroll
                for (int p = 0; p < P; ++p) {
                    const Tail x = tr[s][p], y = ti[s][p];
                    if (k < K) tail = fma_t(w, fma_t(x, x, y * y), tail);
                }
            }
        }
    };

    publish(buf);
    __syncthreads();
    int ppar = 0;
    double fin_norm = 0.0, fin_err = 0.0;
    int alarms = 0, flags = 0;
    for (int64_t step = 0; step < a.steps; ++step) {
        if (sc != 1.0) {   // renormalisation (uniform): rare, so the rows are published again
            const T f = static_cast<T>(sc);
#pragma unroll
            for (int s = 0; s < S; ++s)
#pragma unroll
                for (int p = 0; p < P; ++p) { tr[s][p] *= f; ti[s][p] *= f; }
            __syncthreads();
            publish(buf);
            __syncthreads();
        }
#pragma unroll
        for (int s = 0; s < S; ++s)
#pragma unroll
            for (int p = 0; p < P; ++p) {
                if constexpr (KAHAN) {
                    pr[s][p] = tr[s][p];
                    pi[s][p] = ti[s][p];
                    ar[s][p] = ai[s][p] = T(0);
                } else {
                    ar[s][p] = tr[s][p];
                    ai[s][p] = ti[s][p];
                }
            }
        Tail tail = Tail(0);
        T sgn = T(1);
        T c1 = static_cast<T>(a.coef[1]), c2 = static_cast<T>(a.coef[2]);
        for (int j = 1; j <= n; j += 2) {
            const T d1 = sgn * c1, d2 = -sgn * c2;
            c1 = static_cast<T>(a.coef[j + 2]);   // read while the levels run
            c2 = static_cast<T>(a.coef[j + 3]);
            level(std::true_type{}, d1, j == n, tail);
            if (j < n) level(std::false_type{}, d2, j + 1 == n, tail);
            sgn = -sgn;
        }
        double nrm = 0.0;
        const int kb = here(k0);
#pragma unroll
        for (int s = 0; s < S; ++s) {
            const int k = kb + s;
#pragma unroll
            for (int p = 0; p < P; ++p) {
                if constexpr (KAHAN) {
                    tr[s][p] = pr[s][p] + ar[s][p];
                    ti[s][p] = pi[s][p] + ai[s][p];
                } else {
                    tr[s][p] = ar[s][p];
                    ti[s][p] = ai[s][p];
                }
                if (LAYOUT != kResFull && k >= K) { tr[s][p] = T(0); ti[s][p] = T(0); }
            }
        }
        if constexpr (TRI) {
            // The pairs held twice are rounded differently; the second copy
            // follows the first, so that the state is the stored one after
            // every step and a run cut in two gives the same bits.  (slot_x
            // of the set last read is this wave's alone to read.)
            if (2 * (K - 1) == N && is_top) {
                C* const scratch = pub + (buf * slots + slot_x) * 64 * P;
                const int t = here(top);
                each_slot<S>([&](auto s) {
                    if (t == s) {
                        put(scratch, s);
                        __builtin_amdgcn_wave_barrier();
#pragma unroll
                        for (int p = 0; p < P; ++p) {
                            const int e = lane * P + p - N / 2;
                            if (e >= 0 && in[p]) {
                                const C v = scratch[(e % P) * 64 + e / P];
                                tr[s][p] = v.x;
                                ti[s][p] = v.y;
                            }
                        }
                        own_branch<s>();
                    }
                });
            }
        }
#pragma unroll
        for (int s = 0; s < S; ++s) {
            const int k = kb + s;
            const double w = k < K ? (TRI ? ((k == 0 || 2 * k == N) ? 1.0 : 2.0) : 1.0) : 0.0;
#pragma unroll
            for (int p = 0; p < P; ++p) {
                const double x = tr[s][p], y = ti[s][p];
                nrm = __builtin_fma(w, __builtin_fma(y, y, x * x), nrm);
            }
        }
        nrm = wave_sum_last(nrm);
        const double tl = wave_sum_last((double)tail);
        double* pp = part + ppar * 2 * W;
        if (lane == 63) {
            pp[2 * wv] = nrm;
            pp[2 * wv + 1] = tl;
        }
        publish(buf ^ 1);
        __syncthreads();
        buf ^= 1;
        ppar ^= 1;
        // (every wave when renormalising: the next scale needs the norm)
        if (wv == 0 || a.renormalize) {
            const double ns = lane_value(wave_sum_last(lane < W ? pp[2 * lane] : 0.0), 63);
            const double ts = lane_value(wave_sum_last(lane < W ? pp[2 * lane + 1] : 0.0), 63);
            const double fc = a.coef[n];
            const double err2 = ts * fc * fc * tf * tf;
            fin_norm = ns;
            fin_err = err2;
            int f = 0;
            if (a.tol2 > 0.0 && !(err2 <= a.tol2 * ns)) f |= 1;
            if (!isfinite(ns) || !isfinite(ts)) f |= 2;
            if (a.norm_alarm > 0.0 && !(fabs(sqrt(ns) - 1.0) <= a.norm_alarm)) f |= 2;
            flags |= f;
            alarms += f ? 1 : 0;
            if (a.renormalize) {
                if (ns > 0.0 && isfinite(ns)) sc = 1.0 / sqrt(ns);
            }
        }
        // (without renormalisation a load scale is applied once)
        if (!a.renormalize) sc = 1.0;
        if (a.out_stride > 0 || step + 1 == a.steps) {
            C* out = reinterpret_cast<C*>(reinterpret_cast<char*>(a.psi_out) + step * a.out_stride) + rd.state_off;
            // (the columns anew: kept from the loads, the elements' indices and
            // masks would take registers through the whole run)
            int c0 = lane * P;
            asm volatile("" : "+v"(c0));
#pragma unroll
            for (int s = 0; s < S; ++s)
#pragma unroll
                for (int p = 0; p < P; ++p) {
                    const int e = element(kb, s, c0 + p);
                    if (e >= 0 && (!TRI || 2 * (kb + s) != N || 2 * (c0 + p) < N)) {
                        C v;
                        v.x = tr[s][p];
                        v.y = ti[s][p];
                        out[e] = v;
                    }
                }
        }
    }
    if (threadIdx.x == 0 && a.norm2) {
        a.norm2[r] = fin_norm;
        a.tail2[r] = fin_err;
        if (a.renormalize) a.scale[r] = sc;
        if (flags) {
            atomicOr(&a.status[0], flags);
            atomicAdd(&a.status[1], alarms);
        }
    }
}

template <typename T, int P>
size_t resident_lds(const ResidentShape& s) {
    const bool tri = s.layout == kResTri;
    const int N = s.max_N;
    return 2 * (size_t)(2 * s.waves + 3) * 64 * P * 2 * sizeof(T) + 4 * (size_t)s.waves * sizeof(double) +
           ((tri ? P * bond_plane<P>() : 0) + (size_t)(tri ? N / 2 + 1 : N) * diag_stride<P>(N)) * sizeof(T);
}

}  // namespace resident_detail
}  // namespace ctqw

#define CTQW_RESIDENT(P_, S_, THREADS)                                                                      \
    if (s.cols == P_ && s.rows == S_)                                                                       \
        return {&::ctqw::resident_detail::resident_kernel<T, LAYOUT, P_, S_, KAHAN, THREADS>, THREADS,      \
                &::ctqw::resident_detail::resident_lds<T, P_>};
