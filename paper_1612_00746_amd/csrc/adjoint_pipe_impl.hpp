// The K-level adjoint pass (see adjoint_pipe.hpp for what it computes).
//
// Per wave: one band of columns (one per lane, K halo lanes on either side)
// and one row segment, swept from K rows before the segment to K rows after
// it.  At sweep step i:
//   * level 0: row i of X (or of Z when the pass starts from Z itself)
//     enters, scaled by xs; rows past the sweep enter as zero;
//   * level l = 1 .. K: row i - l of Y_l from level l - 1's rows
//     i - l - 1, i - l, i - l + 1 (a 3-row register window per level), plus
//     cz_l times row i - l of Z; stored if y[l - 1] is set; and, for the
//     Horner passes, level l's input row contracted with rows i - l,
//     i - l + 1 of v[l - 1];
//   * the row parts of row i - K (its last contribution came from level K)
//     join a batch of three rows, which is summed over the wave at once.
// A row's coefficients (and its Z row, its store offsets, its row parts) are
// formed once, as the row enters, and wait in rings of U >= K slots while it
// passes the levels; the sweep is unrolled U rows, so that every slot is a
// compile-time register.  The coefficients are zero wherever no amplitude is
// stored (off the chain, the triangle's lower part, rows past the sweep) and
// hold the triangle's mirrored neighbours on its diagonal, so that a level
// is ten FMAs with nothing to compare or select, and the contractions need
// no masks but those of the finished sums: a lane without a stored amplitude
// multiplies zeros.  The row couplings come through the scalar cache, U rows
// ahead.
//
// Bound, in about equal parts that overlap little, by instruction issue and
// by the vectors' traffic (two bosons, N = 256, 512 realisations, complex64:
// six forward levels take 300 us, of which 140 remain without the stores and
// 140 are the 0.94 GB at a large copy's rate).  Levels that formed their own
// diagonal, masks and offsets took 32 VALU instructions per row and level
// forward and 76 in a Horner pass; these take 15 and 52.  Per time step of
// that gradient (passes of six forward levels and of 3, 2, 2 Horner levels):
// 1070 -> 949 us.  complex128, distinguishable on a ring of 129 sites, 24
// realisations (72 bands): passes of two Horner levels 30 -> 19.6 us, of four
// forward levels 28 -> 18.5 us, where latency is what is left.
//
// Contractions.  Full grid (distinguishable particles; of one particle only the
// column parts): the column parts of bond c and site c are sums over the
// rows, kept per lane; the row parts of bond q and site q are sums over the
// columns, reduced across the wave for three rows at a time into one
// partial per band.
// Bosons are stored as the symmetric function phi(x1, x2) on x1 <= x2; the
// full-grid sums are then twice the column part, and the column part of
// bond b (pairs (q, b), (q, b + 1) over all q) splits into the stored pairs
// of row q <= b in columns b, b + 1 and, mirrored, the pairs of rows b,
// b + 1 in every column c >= b + 1: a horizontal part summed per lane and a
// vertical part summed per row, as for the full grid, with the vertical
// pairs and the row sites taken only where both entries are stored off the
// diagonal (site b: column b over rows q <= b, plus row b over columns
// c > b).  The stencil at a stored diagonal entry (q, q) reads its mirrored
// neighbours (q + 1, q) = (q, q + 1) and (q, q - 1) = (q - 1, q).
#pragma once

#include "adjoint_common.hpp"
#include "adjoint_pipe.hpp"

#include <type_traits>

namespace ctqw {
namespace adj_pipe {

using namespace adj;

__host__ __device__ constexpr int mpos(int x, int w) { return ((x % w) + w) % w; }

// The couplings are read-only while a pass runs: through the scalar cache.
template <typename T>
using ConstPtr = const __attribute__((address_space(4))) T*;

// Coefficients of one row at this lane's column: the level forms
// d m + u (row above) + b (row below) + l (left) + r (right).  u and b are
// per lane for the triangle, whose diagonal mirrors, and uniform otherwise.
//
// complex64 is written out so that the neighbouring columns enter through
// DPP-routed FMAs.  A DPP read of a VGPR must follow the VALU write of that
// register by two wait states: the DPP instructions come after six VALU
// instructions of the block, and their sources are inputs of the block.
//   forward (s = +1): y = -i h;   Horner (s = -1): y = i h.
template <typename T, bool LANE_UB, bool NEG>
__device__ __forceinline__ void stencil(T mr, T mi, T ur, T ui, T dr, T di, T d, T u, T b, T l, T r, T& yr, T& yi,
                                        T& rr, T& ri) {
    if constexpr (sizeof(T) == 4) {
#define CTQW_PIPE_FWD(UB)                                                                    \
    asm("v_mul_f32 %0, %8, %3\n\t"                                                           \
        "v_mul_f32 %1, -%8, %2\n\t"                                                          \
        "v_fma_f32 %0, %9, %5, %0\n\t"                                                       \
        "v_fma_f32 %1, -%9, %4, %1\n\t"                                                      \
        "v_fma_f32 %0, %10, %7, %0\n\t"                                                      \
        "v_fma_f32 %1, -%10, %6, %1\n\t"                                                     \
        "v_fmac_f32_dpp %0, %3, %11 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"  \
        "v_fmac_f32_dpp %1, -%2, %11 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t" \
        "v_fmac_f32_dpp %0, %3, %12 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"  \
        "v_fmac_f32_dpp %1, -%2, %12 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1"     \
        : "=&v"(yr), "=&v"(yi)                                                               \
        : "v"(mr), "v"(mi), "v"(ur), "v"(ui), "v"(dr), "v"(di), "v"(d), UB(u), UB(b), "v"(l), "v"(r))
#define CTQW_PIPE_HORNER(UB)                                                                 \
    asm("v_mul_f32 %0, -%8, %3\n\t"                                                          \
        "v_mul_f32 %1, %8, %2\n\t"                                                           \
        "v_fma_f32 %0, -%9, %5, %0\n\t"                                                      \
        "v_fma_f32 %1, %9, %4, %1\n\t"                                                       \
        "v_fma_f32 %0, -%10, %7, %0\n\t"                                                     \
        "v_fma_f32 %1, %10, %6, %1\n\t"                                                      \
        "v_fmac_f32_dpp %0, -%3, %11 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t" \
        "v_fmac_f32_dpp %1, %2, %11 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"  \
        "v_fmac_f32_dpp %0, -%3, %12 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t" \
        "v_fmac_f32_dpp %1, %2, %12 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1"      \
        : "=&v"(yr), "=&v"(yi)                                                               \
        : "v"(mr), "v"(mi), "v"(ur), "v"(ui), "v"(dr), "v"(di), "v"(d), UB(u), UB(b), "v"(l), "v"(r))
        if constexpr (NEG) {
            if constexpr (LANE_UB) CTQW_PIPE_HORNER("v");
            else CTQW_PIPE_HORNER("s");
        } else {
            if constexpr (LANE_UB) CTQW_PIPE_FWD("v");
            else CTQW_PIPE_FWD("s");
        }
#undef CTQW_PIPE_FWD
#undef CTQW_PIPE_HORNER
    } else {
        rr = from_right(mr);
        ri = from_right(mi);
        const T lr = from_left(mr), li = from_left(mi);
        const T s = NEG ? T(-1) : T(1);
        yr = s * d * mi;
        yi = -s * d * mr;
        yr = fma(s * u, ui, yr);
        yi = fma(-s * u, ur, yi);
        yr = fma(s * b, di, yr);
        yi = fma(-s * b, dr, yi);
        yr = fma(s * l, li, yr);
        yi = fma(-s * l, lr, yi);
        yr = fma(s * r, ri, yr);
        yi = fma(-s * r, rr, yi);
    }
}

// Im conj(y) v with y = a level's input, in the state's precision: the site
// (s0), the bond to the right (hb) and the bond below (vb; d: the input's row
// below, p: v's).  rr, ri: the input's right neighbours (complex128).
template <typename T>
__device__ __forceinline__ void contract(T mr, T mi, T dr, T di, T rr, T ri, T vx, T vy, T px, T py, T& s0, T& hb,
                                         T& vb) {
    if constexpr (sizeof(T) == 4) {
        asm("v_mul_f32 %0, %3, %8\n\t"
            "v_mul_f32 %2, %3, %10\n\t"
            "v_fma_f32 %0, -%4, %7, %0\n\t"
            "v_fma_f32 %2, -%4, %9, %2\n\t"
            "v_fma_f32 %2, %5, %8, %2\n\t"
            "v_fma_f32 %2, -%6, %7, %2\n\t"
            "v_mul_f32_dpp %1, %8, %3 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
            "v_fmac_f32_dpp %1, -%7, %4 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
            "v_fmac_f32_dpp %1, %3, %8 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
            "v_fmac_f32_dpp %1, -%4, %7 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1"
            : "=&v"(s0), "=&v"(hb), "=&v"(vb)
            : "v"(mr), "v"(mi), "v"(dr), "v"(di), "v"(vx), "v"(vy), "v"(px), "v"(py));
    } else {
        const T qx = from_right(vx), qy = from_right(vy);
        s0 = im_t(mr, mi, vx, vy);
        hb = fma(mr, qy, fma(-mi, qx, fma(rr, vy, -(ri * vx))));
        vb = fma(mr, py, fma(-mi, px, fma(dr, vy, -(di * vx))));
    }
}

// One particle: a realisation is a single row, so the levels are K stencils of
// the same lanes and a block is one wave, with every load issued at the start.
// off, off_out: the lane's offset in the row to read and to write (past the end
// where nothing is stored).  As a sweep of 1 + K rows the passes took 3.3 to 4.2
// us in complex128, nearly all of it latency and code fetched once: 259 rings of
// 30 nodes, complex128, 9 steps, 435 -> 367 us per gradient; 66 chains of 242, 418
// -> 360.
template <typename T, int K, bool CON>
__device__ __forceinline__ void one_row(const AdjPipeArgs& a, const RealDev& rd, int r, int cw, bool out, uint32_t off,
                                        uint32_t off_out, T d, T jl, T jr, bool has_bond) {
    using C = typename std::conditional<sizeof(T) == 8, double2, float2>::type;
    auto rsrc = [&](const void* base) {
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<C*>(reinterpret_cast<const C*>(base)) + rd.state_off, 0,
                                                 base ? (int)((uint32_t)rd.N * (uint32_t)sizeof(C)) : 0,
                                                 kRawBufferWord3);
    };
    const C x = load_c(rsrc(a.x), off, (C*)nullptr);
    C z, v[CON ? K : 1];
    double gj = 0.0, ge = 0.0;
    int64_t o = 0;
    if constexpr (CON) {
        z = load_c(rsrc(a.z), off, (C*)nullptr);
#pragma unroll
        for (int l = 0; l < K; ++l) v[l] = load_c(rsrc(a.v[l]), off, (C*)nullptr);
        if (out) {
            o = a.site_off[r] + cw;
            gj = a.gJ[o];
            ge = a.gE[o];
        }
    }
    const T xs = static_cast<T>(a.xs);
    T mr = xs * x.x, mi = xs * x.y;
    double bond = 0.0, site = 0.0;
#pragma unroll
    for (int l = 1; l <= K; ++l) {
        T yr, yi, rr = T(0), ri = T(0);
        stencil<T, false, CON>(mr, mi, T(0), T(0), T(0), T(0), d, T(0), T(0), jl, jr, yr, yi, rr, ri);
        if constexpr (CON) {
            const T cz = static_cast<T>(a.cz[l]);
            yr = fma(cz, z.x, yr);
            yi = fma(cz, z.y, yi);
            T s0, hb, vb;
            contract(mr, mi, T(0), T(0), rr, ri, v[l - 1].x, v[l - 1].y, T(0), T(0), s0, hb, vb);
            site += (double)s0;
            bond += (double)hb;
        }
        if (!CON || l == K) store_c(yr, yi, rsrc(a.y[l - 1]), off_out);
        mr = yr;
        mi = yi;
    }
    if (CON && out) {
        a.gJ[o] = gj + (has_bond ? bond : 0.0);
        a.gE[o] = ge + site;
    }
}

template <typename T, int K, int LAY, bool PER, bool CON>
__global__ void __launch_bounds__(64 * kSweepSegsMax, 2) pipe_kernel(AdjPipeArgs a) {
    using C = typename std::conditional<sizeof(T) == 8, double2, float2>::type;
    constexpr int W = 64 - 2 * K;          // output columns per band
    constexpr int U = 3 * ((K + 2) / 3);   // ring slots and unrolled rows
    static_assert(K >= 1 && K <= kPipeMaxLevels, "levels per pass");
    static_assert(!(PER && LAY == 2), "no triangle on a ring");
    constexpr bool periodic = PER;          // columns on a ring
    constexpr bool rper = PER;              // rows on a ring
    constexpr bool tri = LAY == 2;

    // Consecutive blocks go to the XCDs in turn: a realisation's bands are
    // given to one XCD, whose L2 then holds the halo columns and the lines
    // that two bands share.
    const int r = (int)blockIdx.y * 8 + (blockIdx.x & 7);
    const int w = blockIdx.x >> 3;
    if (r >= a.R) return;   // whole block, before the barrier
    const RealDev rd = a.reals[r];
    const int N = rd.N, rows = rd.rows;
    // Bands are laid from the chain's end: band w outputs [hi - W, hi),
    // hi = N - W (nbr - 1 - w), the first band the rest.
    const int nbr = (N + W - 1) / W;
    if (w >= nbr) return;   // whole block, before the barrier
    const int hi_w = N - W * (nbr - 1 - w);
    const int lo_w = max(0, hi_w - W);
    const int lane = threadIdx.x & 63;
    const int segs = blockDim.x >> 6;   // kSweepSegs or kSweepSegsMax
    const int seg = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const T* Jc = reinterpret_cast<const T*>(a.Jt) + rd.param_off;
    const T* Ec = reinterpret_cast<const T*>(a.Et) + rd.param_off;
    const ConstPtr<T> Jr = (ConstPtr<T>)(reinterpret_cast<uintptr_t>(a.Jt)) + rd.row_param_off;
    const ConstPtr<T> Er = (ConstPtr<T>)(reinterpret_cast<uintptr_t>(a.Et)) + rd.row_param_off;
    const T Udt = static_cast<T>(rd.U * a.dt);
    const int want = (rd.flags & RF_NEAREST) ? 1 : 0;
    const T xs = static_cast<T>(a.xs);

    // this lane's column: window [lo_w - K, lo_w - K + 64), output [lo_w, hi_w)
    const int c = lo_w - K + lane;
    const bool inb = periodic || (c >= 0 && c < N);
    const int cw = periodic ? wrapi(c, N) : (inb ? c : 0);
    const bool out = c >= lo_w && c < hi_w;
    const T jl = (inb && (periodic || c > 0)) ? Jc[periodic ? wrapi(cw - 1, N) : cw - 1] : T(0);
    const T jr = (inb && (periodic || c < N - 1)) ? Jc[cw] : T(0);
    const T ec = inb ? Ec[cw] : T(0);
    const bool has_bond_c = periodic || c < N - 1;
    if constexpr (LAY == 0) {
        const uint32_t off = (uint32_t)cw * (uint32_t)sizeof(C);
        one_row<T, K, CON>(a, rd, r, cw, out, inb ? off : kPastEnd, out ? off : kPastEnd, ec, jl, jr, has_bond_c);
        return;
    }

    // rows holding a stored amplitude of this window, split into one segment
    // per wave; the sweep runs K rows beyond the segment on either side
    const int q_end = tri ? min(rows, hi_w) : rows;
    const int seg_bits = segs == kSweepSegs ? 2 : 3;
    const int q0 = (q_end * seg) >> seg_bits;   // rows < 2^28
    const int q1 = (q_end * (seg + 1)) >> seg_bits;
    const int s_lo = rper ? q0 - K : max(0, q0 - K);
    const int s_hi = rper ? q1 + K : min(rows, q1 + K);
    const int nsweep = q1 > q0 ? s_hi - s_lo : 0;
    const int o_lo = q0 - s_lo, o_hi = q1 - s_lo;   // output rows, as sweep steps

    // One buffer resource per array over this realisation's amplitudes (the
    // launcher keeps them under 2^31 bytes), the row in the per-lane offset:
    // a 32-bit offset per access instead of a resource per row.  Lanes
    // without a stored amplitude (dead), and rows outside a range, take an
    // offset past the end: loads read 0 and stores are dropped.
    const uint32_t col_off = (uint32_t)cw * (uint32_t)sizeof(C);
    const uint32_t dead = inb ? 0u : kPastEnd;
    const uint32_t dead_out = out ? 0u : kPastEnd;
    const uint32_t real_bytes =
        (uint32_t)(tri ? N * (N + 1) / 2 : rows * N) * (uint32_t)sizeof(C);
    auto arr_rsrc = [&](const void* base) {
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<C*>(reinterpret_cast<const C*>(base)) + rd.state_off, 0,
                                                 base ? (int)real_bytes : 0, kRawBufferWord3);
    };
    // offset of grid row q at this lane's column, past the end unless in_row
    auto row_off = [&](int q, bool in_row, uint32_t dead_lanes) -> uint32_t {
        const uint32_t rowb = (uint32_t)(tri ? q * N - (q * (q + 1)) / 2 : q * N) * (uint32_t)sizeof(C);
        const uint32_t base = in_row ? rowb : kPastEnd;
        const uint32_t dl = (tri && cw < q) ? kPastEnd : dead_lanes;
        return (base + col_off) | dl;
    };
    // the next row of the grid (rows past an open grid are never in range)
    auto next_row = [&](int q) { return (rper && q + 1 == rows) ? 0 : q + 1; };

    // The Horner passes (CON) add Z to every level; the forward passes have none.
    const bool x_is_z = CON && a.x == a.z;
    const __amdgpu_buffer_rsrc_t X = arr_rsrc(x_is_z ? nullptr : a.x);
    const __amdgpu_buffer_rsrc_t Z = arr_rsrc(CON ? a.z : nullptr);
    // stored levels: every level of a forward pass, the last of a Horner pass
    __amdgpu_buffer_rsrc_t Y[K], V[CON ? K : 1];
#pragma unroll
    for (int l = 0; l < K; ++l) Y[l] = arr_rsrc((!CON || l == K - 1) ? a.y[l] : nullptr);
    if constexpr (CON) {
#pragma unroll
        for (int l = 0; l < K; ++l) V[l] = arr_rsrc(a.v[l]);
    }

    T yr[K][3], yi[K][3];          // levels 0 .. K - 1, rows modulo 3
    C xq[3], zq[3];                // X and Z rows i .. i + 2, modulo 3
    // rings over the rows in flight, slot = row modulo U
    T cd[U];                       // diagonal
    T cu[tri ? U : 1], cb[tri ? U : 1], cl[tri ? U : 1], cr[tri ? U : 1];
    T sb[U], sb_last = T(0);       // full grid: the bond below the row; sb_last: row i - K - 1's
    uint32_t so[U];                // store offset
    uint32_t vo[CON ? U : 1];      // load offset of v (rows i + 2 .. i + 3 - K)
    T zr[CON ? U : 1], zi[CON ? U : 1];
    T rpv[CON ? U : 1], rps[CON ? U : 1];   // row parts so far
    C vq[CON ? K : 1][3];          // v[l - 1] rows i - l .. i - l + 2, modulo 3
    double batch[8];               // three completed rows (bond, site), two zeros
    T gj[U], ge[U], nj[U], ne[U];  // couplings of this and the next U rows: the bond below, the energy

#pragma unroll
    for (int l = 0; l < K; ++l)
#pragma unroll
        for (int k = 0; k < 3; ++k) yr[l][k] = yi[l][k] = T(0);
#pragma unroll
    for (int k = 0; k < U; ++k) {
        cd[k] = sb[k] = T(0);
        so[k] = kPastEnd;
        if constexpr (tri) cu[k] = cb[k] = cl[k] = cr[k] = T(0);
        if constexpr (CON) {
            vo[k] = kPastEnd;
            zr[k] = zi[k] = rpv[k] = rps[k] = T(0);
        }
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) batch[k] = 0.0;

    const int first = rper ? wrapi(s_lo, rows) : s_lo;
    int qi = first;                // grid row of sweep step i
    int qx = first;                // of step i + 3
    int qn = first;                // of the next group's first row
    const int last = rows - 1;
    auto load_group = [&](T (&j)[U], T (&e)[U]) {
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const int q = min(qn, last);
            j[k] = Jr[q];
            e[k] = Er[q];
            qn = next_row(qn);
        }
    };
    load_group(nj, ne);
    T above = T(0);                // the bond above row i (the row above the sweep holds zeros)
    // rows 0 .. 2 of X and Z, and of v where a level has them in its window
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const uint32_t off = row_off(qx, k < nsweep, dead);
        xq[k] = load_c(X, off, (C*)nullptr);
        if constexpr (CON) {
            zq[k] = load_c(Z, off, (C*)nullptr);
            vo[mpos(k, U)] = row_off(qx, k >= o_lo && k <= o_hi && k < nsweep, dead);
        }
        qx = next_row(qx);
    }
    if constexpr (CON) {
        // level l starts with rows -l .. 2 - l of its v
#pragma unroll
        for (int l = 1; l <= K; ++l)
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                if (k - l >= 0) vq[l - 1][mpos(k - l, 3)] = load_c(V[l - 1], vo[mpos(k - l, U)], (C*)nullptr);
                else vq[l - 1][mpos(k - l, 3)].x = vq[l - 1][mpos(k - l, 3)].y = T(0);
            }
    }
    double bond_col = 0.0, site_col = 0.0;
    const double f = tri ? 2.0 : 1.0;
    // Row sums: lane 8 j holds value j of a batch (rows i - K - 2 .. i - K,
    // bond and site).  Each is read one batch ahead of its addition; a row is
    // in one segment of one band, so no other wave touches it.
    double* g_row = ((lane & 8) ? a.gR : a.gV) + ((int64_t)r * a.nb + w) * a.row_stride;
    const int j_row = lane >> 4;
    auto holds_row = [&](int s) { return (lane & 7) == 0 && j_row < 3 && s >= o_lo && s < o_hi; };
    double g_old = 0.0;
    if (CON) {
        const int s = -K + j_row;
        if (holds_row(s)) g_old = g_row[s_lo + s];
    }

    const int total = nsweep > 0 ? nsweep + K : 0;
    for (int i0 = 0; i0 < total; i0 += U) {
#pragma unroll
        for (int k = 0; k < U; ++k) {
            gj[k] = nj[k];
            ge[k] = ne[k];
        }
        load_group(nj, ne);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = i0 + u;
            // ---- level 0: row i enters (past the sweep the loads gave zero)
            const C xv = (CON && x_is_z) ? zq[mpos(u, 3)] : xq[mpos(u, 3)];
            yr[0][mpos(u, 3)] = xs * xv.x;
            yi[0][mpos(u, 3)] = xs * xv.y;
            const C zv = zq[mpos(u, 3)];
            const uint32_t xo = row_off(qx, i + 3 < nsweep, dead);
            xq[mpos(u, 3)] = load_c(X, xo, (C*)nullptr);
            if constexpr (CON) zq[mpos(u, 3)] = load_c(Z, xo, (C*)nullptr);
            // ---- levels 1 .. K: row s = i - l
#pragma unroll
            for (int l = 1; l <= K; ++l) {
                const int s = i - l;
                const int su = mpos(u - l - 1, 3), sm = mpos(u - l, 3), sd = mpos(u - l + 1, 3);
                const int slot = mpos(u - l, U);
                const T mr = yr[l - 1][sm], mi = yi[l - 1][sm];
                const T ur_ = yr[l - 1][su], ui_ = yi[l - 1][su];   // row s - 1
                const T dr_ = yr[l - 1][sd], di_ = yi[l - 1][sd];   // row s + 1
                T yr_, yi_, rr = T(0), ri = T(0);
                if constexpr (tri) {
                    stencil<T, true, CON>(mr, mi, ur_, ui_, dr_, di_, cd[slot], cu[slot], cb[slot], cl[slot],
                                          cr[slot], yr_, yi_, rr, ri);
                } else {
                    const T up = (U == K && l == K) ? sb_last : sb[mpos(u - l - 1, U)];
                    stencil<T, false, CON>(mr, mi, ur_, ui_, dr_, di_, cd[slot], up, sb[slot], jl, jr, yr_, yi_, rr,
                                           ri);
                }
                if constexpr (CON) {
                    // last: Z outweighs the rest, which would round at its size
                    const T cz = static_cast<T>(a.cz[l]);
                    yr_ = fma(cz, zr[slot], yr_);
                    yi_ = fma(cz, zi[slot], yi_);
                }
                if (!CON || l == K) store_c(yr_, yi_, Y[l - 1], so[slot]);
                if constexpr (CON) {
                    const C v0 = vq[l - 1][sm], vp = vq[l - 1][sd];
                    T s0, hb, vb;
                    contract(mr, mi, dr_, di_, rr, ri, v0.x, v0.y, vp.x, vp.y, s0, hb, vb);
                    rpv[slot] += vb;
                    rps[slot] += s0;
                    // rows of the segment only; v holds zeros before it
                    const double own = (s >= o_lo && s < o_hi) ? 1.0 : 0.0;
                    site_col = fma(own, (double)s0, site_col);
                    bond_col = fma(own, (double)hb, bond_col);
                    // v[l - 1] row s + 3
                    vq[l - 1][sm] = load_c(V[l - 1], vo[mpos(u - l + 3, U)], (C*)nullptr);
                }
                if (l < K) {
                    yr[l][sm] = yr_;
                    yi[l][sm] = yi_;
                }
            }
            if constexpr (CON) {
                // row i - K is complete; its slot takes row i
                const bool diag = tri && cw == qi - K;
                batch[2 * mpos(u, 3)] = (double)(out ? rpv[mpos(u - K, U)] : T(0));
                batch[2 * mpos(u, 3) + 1] = (double)((out && !diag) ? rps[mpos(u - K, U)] : T(0));
                if (mpos(u, 3) == 2) {
                    // lane 8 j ends with the wave's sum of batch[j]
                    const double t = reduce8(batch, lane);
                    const int sr = i - K - 2 + j_row;
                    if (holds_row(sr)) g_row[s_lo + sr] = g_old + f * t;
                    if (holds_row(sr + 3)) g_old = g_row[s_lo + sr + 3];
                }
                vo[mpos(u + 3, U)] = row_off(qx, i + 3 >= o_lo && i + 3 <= o_hi && i + 3 < nsweep, dead);
            }
            // ---- row i's coefficients take the slot
            {
                const bool live = i < nsweep;
                const bool stored = inb && (!tri || cw >= qi);
                int dd = qi - cw;
                dd = dd < 0 ? -dd : dd;
                if (periodic && N - dd < dd) dd = N - dd;
                T d = ge[u] + ec;
                if (dd == want) d += Udt;
                cd[mpos(u, U)] = (live && stored) ? d : T(0);
                // the bond to row i + 1: none below the grid or past the sweep
                const T below = i + 1 < nsweep ? gj[u] : T(0);
                if constexpr (tri) {
                    const bool diag = cw == qi;
                    cu[mpos(u, U)] = stored ? (diag ? above + jl : above) : T(0);
                    cb[mpos(u, U)] = (stored && !diag) ? below : T(0);
                    cl[mpos(u, U)] = (stored && !diag) ? jl : T(0);
                    cr[mpos(u, U)] = stored ? (diag ? jr + below : jr) : T(0);
                    above = below;
                } else {
                    if (U == K) sb_last = sb[mpos(u, U)];
                    sb[mpos(u, U)] = below;
                }
                so[mpos(u, U)] = row_off(qi, i >= o_lo && i < o_hi, dead | dead_out);
                if constexpr (CON) {
                    zr[mpos(u, U)] = zv.x;
                    zi[mpos(u, U)] = zv.y;
                    rpv[mpos(u, U)] = rps[mpos(u, U)] = T(0);
                }
            }
            qi = next_row(qi);
            qx = next_row(qx);
            __builtin_amdgcn_sched_barrier(0);   // rows interleaved would not fit the registers
        }
    }
    if constexpr (CON) {
        // column parts of the segments, summed in segment order
        __shared__ double part[2][kSweepSegsMax][64];
        part[0][seg][lane] = has_bond_c ? bond_col : 0.0;
        part[1][seg][lane] = site_col;
        __syncthreads();
        if (seg == 0 && out) {
            double sb = 0.0, ss = 0.0;
            for (int k = 0; k < segs; ++k) {
                sb += part[0][k][lane];
                ss += part[1][k][lane];
            }
            const int64_t o = a.site_off[r] + cw;
            a.gJ[o] += f * sb;
            a.gE[o] += f * ss;
        }
    }
}

}  // namespace adj_pipe
}  // namespace ctqw
