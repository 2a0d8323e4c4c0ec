// One particle on a two-dimensional lattice (q = 2: Sec. 2, a node couples to
// its four lattice neighbours; the capacity example of Sec. 3), R statically
// noisy realisations, each with its own coupling on every bond and its own
// on-site energy on every node (Eq. 1 with the noise drawn per bond and per
// node), advanced by the truncated Taylor series of exp(-i H dt) (Eqs. 5-7,
// Alg. 3) with all n terms of a step in one pass over the state.
//
// The state of realisation r is psi[r][y][x] (x fastest).  A work item is a
// band of 64 P columns (P per lane: two for complex64, one for complex128 and
// narrow lattices) of one realisation, or a segment of its rows, swept over
// the rows y with an n-level register pipeline: at sweep step i row i enters
// level 0, level j completes Y_j = (dt H) Y_(j-1) on row i - j when level j - 1
// hands it row i - j + 1, and row i - n is complete.
//   (dt H y)(x, y) = jd(x, y - 1) u + e(x, y) m + jr(x - 1, y) l + jr(x, y) r + jd(x, y) d
// (m: this amplitude; u, d: the rows above and below; l, r: the adjacent
// columns).  The products are summed as their rows arrive -- a level holds
// the started sum of one row and the product the next row starts from, two
// rows instead of a window of three -- and the tables, which vary along both
// axes, ride in a ring of rows in LDS private to the wave (dt-scaled as they
// are read), so that two columns per lane at 10 terms fit two waves per SIMD.
// The terms (-i)^j Y_j / j! are summed apart from psi and added to it once,
// when the row completes; the squared FP64 norm of the new state is reduced
// per item.  Bands overlap by n columns (the halo); a ring in y, and a
// segment of rows, are swept n rows early and late.
//
// HBM bytes per node and step: read psi and the three tables, write psi
// (complex64: 8 + 12 + 8 = 28 B), times the band overlap on the reads.
// Bound by the vector ALUs' issue (about 28 instructions per level and 128
// columns).  128 x 128, 4096 realisations, 10 terms, us per step, with one
// column per lane, the tables in registers and three-row windows -> now:
// complex64 668 -> 409 (4.6 TB/s), complex128 1286 -> 997.
#include "../../include/ctqw.h"
#include "ctqw_internal.hpp"

#include <algorithm>
#include <vector>

namespace ctqw {
namespace lattice_detail {

template <typename T> struct Cplx;
template <> struct Cplx<float> { using type = float2; };
template <> struct Cplx<double> { using type = double2; };

typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
constexpr int kWord3 = 0x00020000;            // gfx9-family raw buffer, no format conversion
constexpr uint32_t kPastEnd = 0x80000000u;    // an offset past every row: loads read 0, stores drop

__device__ __forceinline__ float lane_left(float x) { return __builtin_amdgcn_update_dpp(0.0f, x, 0x138, 0xF, 0xF, true); }
__device__ __forceinline__ double lane_left(double x) { return __builtin_amdgcn_update_dpp(0.0, x, 0x138, 0xF, 0xF, true); }
__device__ __forceinline__ float lane_right(float x) { return __builtin_amdgcn_update_dpp(0.0f, x, 0x130, 0xF, 0xF, true); }
__device__ __forceinline__ double lane_right(double x) { return __builtin_amdgcn_update_dpp(0.0, x, 0x130, 0xF, 0xF, true); }

__device__ __forceinline__ float fmat(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double fmat(double a, double b, double c) { return __builtin_fma(a, b, c); }

__device__ __forceinline__ float2 load_c(__amdgpu_buffer_rsrc_t rs, uint32_t off, float2*) {
    const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(rs, (int)off, 0, 0);
    return make_float2(__uint_as_float(v.x), __uint_as_float(v.y));
}
__device__ __forceinline__ double2 load_c(__amdgpu_buffer_rsrc_t rs, uint32_t off, double2*) {
    const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rs, (int)off, 0, 0);
    return make_double2(__hiloint2double((int)v.y, (int)v.x), __hiloint2double((int)v.w, (int)v.z));
}
__device__ __forceinline__ float load_r(__amdgpu_buffer_rsrc_t rs, uint32_t off, float*) {
    return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, (int)off, 0, 0));
}
__device__ __forceinline__ double load_r(__amdgpu_buffer_rsrc_t rs, uint32_t off, double*) {
    const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(rs, (int)off, 0, 0);
    return __hiloint2double((int)v.y, (int)v.x);
}
// Stores take a zero scalar offset (a 16-byte store reads its data registers
// after it issues; the compiler keeps the wait before the next write of
// them only when the scalar offset is not a register).
__device__ __forceinline__ void store_c(float re, float im, __amdgpu_buffer_rsrc_t rs, uint32_t off) {
    u32x2 v;
    v.x = __float_as_uint(re);
    v.y = __float_as_uint(im);
    __builtin_amdgcn_raw_buffer_store_b64(v, rs, (int)off, 0, 2);
}
__device__ __forceinline__ void store_c(double re, double im, __amdgpu_buffer_rsrc_t rs, uint32_t off) {
    u32x4 v;
    v.x = (unsigned)__double2loint(re);
    v.y = (unsigned)__double2hiint(re);
    v.z = (unsigned)__double2loint(im);
    v.w = (unsigned)__double2hiint(im);
    __builtin_amdgcn_raw_buffer_store_b128(v, rs, (int)off, 0, 2);
}

// Rows of the ring, the unrolled block of a sweep: those in flight, n levels
// and the row entering; even, so that the rows being fetched (two) divide it.
// A sweep runs whole blocks (leaving one early would cost every block a branch
// that its registers have to meet at: 5 to 15 % of a long sweep), so short ones
// may run mostly past their end.  At the orders where the registers and the LDS
// keep their waves there is a second ring of two rows more, for the sweeps that
// it covers in fewer rows (us per 8 steps, first ring -> chosen by itself, and
// the three-row sweeps before; complex128 unless said): 33 x 13, 8 terms, 21 rows
// in 30 or 24: 170 -> 145 (141); 163 x 12, 6 terms, 18 in 24 or 20: 126 -> 113
// (108); 249 x 15, 9 terms, 24 in 30 or 24: 187 -> 160 (161); complex64 15 x 15,
// 8 terms: 140 -> 119 (128); 171 x 4, 1748 realisations, 8 terms: 493 -> 330
// (445).
constexpr int kWideFrom = 4, kWideTo = 9;   // orders of the second ring
__host__ __device__ constexpr int ring_rows(int nt, bool wide) { return ((nt + 2) & ~1) + (wide ? 2 : 0); }
// rows that a sweep of `rows` runs with a ring, and whether the second's are fewer
inline int64_t swept_rows(int64_t rows, int nt, bool wide) {
    const int64_t block = ring_rows(nt, wide);
    return (rows + block - 1) / block * block;
}
inline bool wide_ring(int64_t rows, int nt) {
    return nt >= kWideFrom && nt <= kWideTo && swept_rows(rows, nt, true) < swept_rows(rows, nt, false);
}
__host__ __device__ constexpr int mpos(int x, int w) { return ((x % w) + w) % w; }
__host__ __device__ constexpr double inv_fact(int j) {
    double f = 1.0;
    for (int k = 2; k <= j; ++k) f *= k;
    return 1.0 / f;
}
// (-i)^j = (sr, si) applied after the swap of roles: for odd j the real part
// of (-i)^j y is si_j Im y, the imaginary part sr_j Re y.
__host__ __device__ constexpr double rot_re(int j) { return (j % 4 == 0 || j % 4 == 1) ? 1.0 : -1.0; }
__host__ __device__ constexpr double rot_im(int j) { return (j % 4 == 0 || j % 4 == 3) ? 1.0 : -1.0; }

// Band b of W columns with a halo of h: window start w0, output [lo, hi).
// Open chain: the first window starts at column 0 and every later one h
// columns before its output; a window that reaches the end outputs up to
// it.  Ring: every window starts h columns before its output.
__host__ __device__ inline void band_geom(int b, int Lx, int h, bool periodic, int* w0, int* lo, int* hi, int W = 64) {
    const int step = W - 2 * h;
    if (periodic) {
        *lo = b * step;
        *w0 = *lo - h;
        *hi = (*lo + step < Lx) ? *lo + step : Lx;
    } else {
        *lo = b == 0 ? 0 : W - h + (b - 1) * step;
        *w0 = b == 0 ? 0 : *lo - h;
        *hi = (*w0 + W >= Lx) ? Lx : *w0 + W - h;
    }
}
// Bands up to the one whose output reaches the end of the chain.
__host__ inline int band_count(int Lx, int h, bool periodic, int W = 64) {
    if (W - 2 * h <= 0) return 0;
    for (int b = 0;; ++b) {
        int w0, lo, hi;
        band_geom(b, Lx, h, periodic, &w0, &lo, &hi, W);
        if (hi >= Lx) return b + 1;
    }
}
// Halo of a band: the terms, at two columns per lane rounded up to even (the
// lanes' column pairs then start on even columns).
__host__ __device__ constexpr int halo_of(int nt, int cols) { return cols == 2 ? (nt + 1) & ~1 : nt; }

__device__ __forceinline__ int wrapi(int x, int n) { int r = x % n; return r < 0 ? r + n : r; }

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// One lane's P values of a row of a table or of the state.  VEC: the lane's
// two columns are adjacent in memory, both on the chain or both off it, and
// 16-byte aligned pairs (the host checks), one access.
template <typename T, int P, bool VEC>
__device__ __forceinline__ void load_row(__amdgpu_buffer_rsrc_t rs, const uint32_t (&off)[P], T (&re)[P], T (&im)[P]) {
    using C = typename Cplx<T>::type;
    if constexpr (VEC) {
        static_assert(P == 2 && sizeof(T) == 4, "pairs of complex64");
        const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rs, (int)off[0], 0, 0);
        re[0] = __uint_as_float(v.x);
        im[0] = __uint_as_float(v.y);
        re[P - 1] = __uint_as_float(v.z);
        im[P - 1] = __uint_as_float(v.w);
    } else {
#pragma unroll
        for (int p = 0; p < P; ++p) {
            const C v = load_c(rs, off[p], (C*)nullptr);
            re[p] = v.x;
            im[p] = v.y;
        }
    }
}
template <typename T, int P, bool VEC>
__device__ __forceinline__ void load_tab(__amdgpu_buffer_rsrc_t rs, const uint32_t (&off)[P], T (&x)[P]) {
    if constexpr (VEC) {
        const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(rs, (int)off[0], 0, 0);
        x[0] = __uint_as_float(v.x);
        x[P - 1] = __uint_as_float(v.y);
    } else {
#pragma unroll
        for (int p = 0; p < P; ++p) x[p] = load_r(rs, off[p], (T*)nullptr);
    }
}

// One level of the pipeline for a lane's P columns.  x: the row handed down,
// Y_(j-1) on row q + 1; e, jr, jl, d: that row's energies, bonds right and left
// of the lane's first column and bonds below; b: the bonds below row q; s: row
// q's sum so far, then row q + 1's; u: what row q + 1, then q + 2, starts
// from; y: Y_j on row q.
//   y = s + b x;  s = u + e x + (left) + (right);  u = d x
// complex64 is written out so that the adjacent lanes' columns enter through
// DPP-routed FMAs (25 instead of 29 instructions per level and lane pair: 456
// instead of 470 us per step of the 128 x 128 batch above).  A DPP read of a VGPR must follow the VALU write of that register by
// two wait states: the DPP instructions come after six VALU instructions of
// the block, and their sources are inputs of the block.
template <typename T, int P>
__device__ __forceinline__ void level(const T (&xr)[P], const T (&xi)[P], const T (&e)[P], const T (&jr)[P], T jl,
                                      const T (&d)[P], const T (&b)[P], T (&sr)[P], T (&si)[P], T (&ur)[P], T (&ui)[P],
                                      T (&yr)[P], T (&yi)[P]) {
    if constexpr (sizeof(T) == 4 && P == 2) {
        asm("v_fma_f32 %0, %20, %12, %4\n\t"
            "v_fma_f32 %1, %20, %13, %5\n\t"
            "v_fma_f32 %2, %21, %14, %6\n\t"
            "v_fma_f32 %3, %21, %15, %7\n\t"
            "v_fma_f32 %4, %16, %12, %8\n\t"
            "v_fma_f32 %5, %16, %13, %9\n\t"
            "v_fma_f32 %6, %17, %14, %10\n\t"
            "v_fma_f32 %7, %17, %15, %11\n\t"
            "v_mul_f32 %8, %22, %12\n\t"
            "v_mul_f32 %9, %22, %13\n\t"
            "v_mul_f32 %10, %23, %14\n\t"
            "v_mul_f32 %11, %23, %15\n\t"
            "v_fmac_f32_dpp %4, %14, %24 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
            "v_fmac_f32_dpp %5, %15, %24 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
            "v_fmac_f32 %6, %18, %12\n\t"
            "v_fmac_f32 %7, %18, %13\n\t"
            "v_fmac_f32 %4, %18, %14\n\t"
            "v_fmac_f32 %5, %18, %15\n\t"
            "v_fmac_f32_dpp %6, %12, %19 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
            "v_fmac_f32_dpp %7, %13, %19 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1"
            : "=&v"(yr[0]), "=&v"(yi[0]), "=&v"(yr[1]), "=&v"(yi[1]), "+&v"(sr[0]), "+&v"(si[0]), "+&v"(sr[1]),
              "+&v"(si[1]), "+&v"(ur[0]), "+&v"(ui[0]), "+&v"(ur[1]), "+&v"(ui[1])
            : "v"(xr[0]), "v"(xi[0]), "v"(xr[1]), "v"(xi[1]), "v"(e[0]), "v"(e[1]), "v"(jr[0]), "v"(jr[1]), "v"(b[0]),
              "v"(b[1]), "v"(d[0]), "v"(d[1]), "v"(jl));
    } else if constexpr (sizeof(T) == 4) {
        asm("v_fma_f32 %0, %10, %6, %2\n\t"
            "v_fma_f32 %1, %10, %7, %3\n\t"
            "v_fma_f32 %2, %8, %6, %4\n\t"
            "v_fma_f32 %3, %8, %7, %5\n\t"
            "v_mul_f32 %4, %11, %6\n\t"
            "v_mul_f32 %5, %11, %7\n\t"
            "v_fmac_f32_dpp %2, %6, %12 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
            "v_fmac_f32_dpp %3, %7, %12 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
            "v_fmac_f32_dpp %2, %6, %9 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
            "v_fmac_f32_dpp %3, %7, %9 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1"
            : "=&v"(yr[0]), "=&v"(yi[0]), "+&v"(sr[0]), "+&v"(si[0]), "+&v"(ur[0]), "+&v"(ui[0])
            : "v"(xr[0]), "v"(xi[0]), "v"(e[0]), "v"(jr[0]), "v"(b[0]), "v"(d[0]), "v"(jl));
    } else {
        T lr[P], li[P], rr[P], ri[P], jleft[P];
        lr[0] = lane_left(xr[P - 1]);
        li[0] = lane_left(xi[P - 1]);
        jleft[0] = jl;
        rr[P - 1] = lane_right(xr[0]);
        ri[P - 1] = lane_right(xi[0]);
#pragma unroll
        for (int p = 0; p + 1 < P; ++p) {
            lr[p + 1] = xr[p];
            li[p + 1] = xi[p];
            jleft[p + 1] = jr[p];
            rr[p] = xr[p + 1];
            ri[p] = xi[p + 1];
        }
#pragma unroll
        for (int p = 0; p < P; ++p) {
            yr[p] = fmat(b[p], xr[p], sr[p]);
            yi[p] = fmat(b[p], xi[p], si[p]);
            T hr = fmat(e[p], xr[p], ur[p]);
            T hi = fmat(e[p], xi[p], ui[p]);
            hr = fmat(jleft[p], lr[p], hr);
            hi = fmat(jleft[p], li[p], hi);
            sr[p] = fmat(jr[p], rr[p], hr);
            si[p] = fmat(jr[p], ri[p], hi);
            ur[p] = d[p] * xr[p];
            ui[p] = d[p] * xi[p];
        }
    }
}

// LDS of one wave: a ring of table rows, {e, jr} and {jd} of every lane.
template <typename T, int P>
constexpr size_t wave_lds(int ring) { return (size_t)ring * 64 * 3 * P * sizeof(T); }

template <typename T, int NT, int P, bool VEC, int WA>
__global__ void __launch_bounds__(256, 2) lattice_kernel(LatticeArgs a) {
    using C = typename Cplx<T>::type;
    constexpr int W = 64 * P, H = halo_of(NT, P);
    constexpr int PF = 2;   // rows fetched ahead
    // complex128: the bonds to the left shifted once per row instead of in every
    // level (two moves of 28 instructions) where the ring of them costs no wave
    // per SIMD (13 x 56, 4190 realisations, 6 terms, 8 steps: 831 -> 796 us;
    // order 5 would fall from three waves to two and take 10 % more)
    constexpr bool KEEPL = sizeof(T) == 8 && NT >= 4 && NT <= 8 && NT != 5;
    constexpr int AHEAD = P == 2 ? 1 : (sizeof(T) == 4 ? 3 : 2);   // levels whose tables are read ahead
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int item = (int)blockIdx.x * 4 + wv;
    if (item >= a.n_items) return;   // whole wave; the kernel has no barrier
    const int seg = __builtin_amdgcn_readfirstlane(item % a.segs);
    const int rb = __builtin_amdgcn_readfirstlane(item / a.segs);
    const int r = __builtin_amdgcn_readfirstlane(rb / a.nb);
    const int b = __builtin_amdgcn_readfirstlane(rb % a.nb);
    const int Lx = a.Lx, Ly = a.Ly;
    const bool px = a.px != 0, py = a.py != 0;
    int w0, lo, hi;
    band_geom(b, Lx, H, px, &w0, &lo, &hi, W);
    const int64_t nodes = (int64_t)Lx * Ly;

    extern __shared__ char lds_raw[];
    struct alignas(2 * P * sizeof(T)) EJ { T e[P], jr[P]; };
    struct alignas(P * sizeof(T)) JD { T d[P]; };
    EJ* const ring_ej = reinterpret_cast<EJ*>(lds_raw + wv * wave_lds<T, P>(WA)) + lane;
    JD* const ring_jd = reinterpret_cast<JD*>(lds_raw + wv * wave_lds<T, P>(WA) + (size_t)WA * 64 * sizeof(EJ)) + lane;

    // this lane's columns (an open axis has no bond past its last node)
    bool outv[P];
    uint32_t off_c[P], off_t[P], off_j[P], off_o[P];
#pragma unroll
    for (int p = 0; p < P; ++p) {
        const int c = w0 + lane * P + p;
        const bool inb = px || (c >= 0 && c < Lx);
        const int cw = px ? wrapi(c, Lx) : (inb ? c : 0);
        outv[p] = inb && c >= lo && c < hi;
        off_c[p] = inb ? (uint32_t)cw * (uint32_t)sizeof(C) : kPastEnd;
        off_t[p] = inb ? (uint32_t)cw * (uint32_t)sizeof(T) : kPastEnd;
        off_j[p] = (inb && (px || c < Lx - 1)) ? off_t[p] : kPastEnd;
        off_o[p] = outv[p] ? (uint32_t)cw * (uint32_t)sizeof(C) : kPastEnd;
    }
    // (a pair of bonds read at once: the one past the end is dropped below)
    const bool last_pair = VEC && !px && w0 + lane * P + P - 1 == Lx - 1;

    const C* in = static_cast<const C*>(a.psi_in) + r * nodes;
    C* out = static_cast<C*>(a.psi_out) + r * nodes;
    const T* jx = static_cast<const T*>(a.Jx) + r * nodes;
    const T* jy = static_cast<const T*>(a.Jy) + r * nodes;
    const T* es = static_cast<const T*>(a.eps) + r * nodes;
    const T dt = static_cast<T>(a.dt);
    // output rows of the segment, and the rows swept for them
    const int out_lo = (int)((int64_t)Ly * seg / a.segs), out_hi = (int)((int64_t)Ly * (seg + 1) / a.segs);
    const bool whole = a.segs == 1 && !py;
    const int row0 = whole ? 0 : (py ? out_lo - NT : max(0, out_lo - NT));
    const int nrows = (whole ? Ly : (py ? out_hi + NT : min(Ly, out_hi + NT))) - row0;
    const uint32_t row_c = (uint32_t)Lx * (uint32_t)sizeof(C);
    const uint32_t row_t = (uint32_t)Lx * (uint32_t)sizeof(T);

    // Row i of the sweep through buffer resources (length 0 past the sweep,
    // and for the bonds below an open axis's last row).
    T fr[PF][P], fi[PF][P], fj[PF][P], fd[PF][P], fe[PF][P];
    int qf = py ? wrapi(row0, Ly) : row0;   // row fetched next
    auto fetch = [&](int i, int slot) {
        const bool live = i < nrows;
        const int64_t base = (int64_t)(live ? qf : 0) * Lx;
        auto rsrc = [&](const void* p, uint32_t bytes) {
            return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)bytes, kWord3);
        };
        load_row<T, P, VEC>(rsrc(in + base, live ? row_c : 0), off_c, fr[slot], fi[slot]);
        load_tab<T, P, VEC>(rsrc(jx + base, live ? row_t : 0), VEC ? off_t : off_j, fj[slot]);
        load_tab<T, P, VEC>(rsrc(jy + base, live && (py || qf < Ly - 1) ? row_t : 0), off_t, fd[slot]);
        load_tab<T, P, VEC>(rsrc(es + base, live ? row_t : 0), off_t, fe[slot]);
        qf = (qf + 1 == Ly) ? 0 : qf + 1;
    };

    T sr[NT][P], si[NT][P];             // level j: its row's sum so far (all but the row below)
    T ur[NT][P], ui[NT][P];             // level j: what its next row starts from
    T pr[WA][P], pi[WA][P];             // psi of the rows in flight
    T tr[WA][P], ti[WA][P];             // their summed terms
    T lr[KEEPL ? WA : 1];               // the bonds to the left of their first columns
#pragma unroll
    for (int p = 0; p < P; ++p) {
#pragma unroll
        for (int j = 0; j < NT; ++j) sr[j][p] = si[j][p] = ur[j][p] = ui[j][p] = T(0);
#pragma unroll
        for (int w = 0; w < WA; ++w) pr[w][p] = pi[w][p] = tr[w][p] = ti[w][p] = T(0);
    }
#pragma unroll
    for (int w = 0; w < (KEEPL ? WA : 1); ++w) lr[w] = T(0);
    {
        EJ z{};
        JD zd{};
#pragma unroll
        for (int w = 0; w < WA; ++w) {
            ring_ej[w * 64] = z;
            ring_jd[w * 64] = zd;
        }
    }
#pragma unroll
    for (int s = 0; s < PF; ++s) {
        fetch(s, s);
        __builtin_amdgcn_sched_barrier(0);
    }

    double nrm = 0.0;
    const int total = nrows + NT;
    static_assert(WA % PF == 0, "the fetched rows must divide the unrolled block");
    for (int i0 = 0; i0 < total; i0 += WA) {
#pragma unroll
        for (int u = 0; u < WA; ++u) {
            const int i = i0 + u;
            const int w = u, sp = u % PF;
            // ---- level 0: row i enters (zero past the sweep)
            T xr[P], xi[P];             // the row handed down, Y_(j-1) on row i - j + 1
            EJ ej;                      // its tables
            JD jd;
#pragma unroll
            for (int p = 0; p < P; ++p) {
                xr[p] = pr[w][p] = fr[sp][p];
                xi[p] = pi[w][p] = fi[sp][p];
                tr[w][p] = ti[w][p] = T(0);
                ej.e[p] = dt * fe[sp][p];
                ej.jr[p] = dt * fj[sp][p];
                jd.d[p] = dt * fd[sp][p];
            }
            if (VEC) ej.jr[P - 1] = last_pair ? T(0) : ej.jr[P - 1];
            if (KEEPL) lr[w] = lane_left(ej.jr[P - 1]);
            fetch(i + PF, sp);
            // tables of the next AHEAD levels' rows (of row i - j: te, the bonds
            // below it: td), read while the levels before them run: a level of
            // one column per lane is shorter than the read
            EJ te[AHEAD];
            JD td[AHEAD];
            auto read = [&](int j) {
                if (j < NT) te[j % AHEAD] = ring_ej[mpos(u - j, WA) * 64];
                if (j <= NT) td[j % AHEAD] = ring_jd[mpos(u - j, WA) * 64];
            };
#pragma unroll
            for (int j = 1; j <= AHEAD; ++j) read(j);
            ring_ej[w * 64] = ej;
            ring_jd[w * 64] = jd;
            // ---- levels 1..NT: row i - j completes, row i - j + 1 starts
#pragma unroll
            for (int j = 1; j <= NT; ++j) {
                const int wj = mpos(u - j, WA);
                const JD below = td[j % AHEAD];
                const EJ ej_next = te[j % AHEAD];
                read(j + AHEAD);
                __builtin_amdgcn_sched_barrier(0);
                const T jl = KEEPL ? lr[KEEPL ? mpos(u - j + 1, WA) : 0] : lane_left(ej.jr[P - 1]);
                const T cr = static_cast<T>(rot_re(j) * inv_fact(j)), ci = static_cast<T>(rot_im(j) * inv_fact(j));
                T yr[P], yi[P];
                level<T, P>(xr, xi, ej.e, ej.jr, jl, jd.d, below.d, sr[j - 1], si[j - 1], ur[j - 1], ui[j - 1], yr, yi);
#pragma unroll
                for (int p = 0; p < P; ++p) {
                    // (-i)^j Y_j / j!: odd j swaps the parts
                    tr[wj][p] = fmat(cr, (j & 1) ? yi[p] : yr[p], tr[wj][p]);
                    ti[wj][p] = fmat(ci, (j & 1) ? yr[p] : yi[p], ti[wj][p]);
                    xr[p] = yr[p];
                    xi[p] = yi[p];
                }
                jd = below;
                if (j < NT) ej = ej_next;
            }
            // ---- row i - NT is complete
            {
                const int wo = mpos(u - NT, WA);
                const int qa = row0 + i - NT;
                const bool ok = qa >= out_lo && qa < out_hi;
                const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
                    out + (int64_t)(ok ? qa : 0) * Lx, 0, ok ? (int)row_c : 0, kWord3);
                T orr[P], oi[P];
#pragma unroll
                for (int p = 0; p < P; ++p) {
                    orr[p] = pr[wo][p] + tr[wo][p];
                    oi[p] = pi[wo][p] + ti[wo][p];
                    const double dr = orr[p], di = oi[p];
                    const double s = __builtin_fma(dr, dr, __builtin_fma(di, di, nrm));
                    nrm = (ok && outv[p]) ? s : nrm;
                }
                if constexpr (VEC) {
                    u32x4 v;
                    v.x = __float_as_uint(orr[0]);
                    v.y = __float_as_uint(oi[0]);
                    v.z = __float_as_uint(orr[P - 1]);
                    v.w = __float_as_uint(oi[P - 1]);
                    __builtin_amdgcn_raw_buffer_store_b128(v, rs, (int)off_o[0], 0, 2);
                } else {
#pragma unroll
                    for (int p = 0; p < P; ++p) store_c(orr[p], oi[p], rs, off_o[p]);
                }
            }
            __builtin_amdgcn_sched_barrier(0);   // one row's work at a time
        }
    }
    nrm = wave_sum(nrm);
    if (lane == 0) a.norm_part[item] = nrm;
}

// out[k][r] = sum over the items of realisation r in step k of their
// partials, in item order.
__global__ void lattice_norm_kernel(const double* part, int32_t per, int32_t R, int32_t steps, double* out) {
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= (int64_t)R * steps) return;
    double s = 0.0;
    for (int b = 0; b < per; ++b) s += part[k * per + b];
    out[k] = s;
}

struct Kernel {
    void (*fn)(LatticeArgs) = nullptr;
    size_t lds = 0;
};
template <typename T, int NT, int P, bool VEC, bool WIDE>
Kernel kernel_of() {
    constexpr int WA = ring_rows(NT, WIDE);
    return Kernel{&lattice_kernel<T, NT, P, VEC, WA>, 4 * wave_lds<T, P>(WA)};
}
template <typename T, int P, bool VEC, int... Ns>
Kernel pick(int order, std::integer_sequence<int, Ns...>) {
    Kernel k;
    ((k = (order == Ns + 1) ? kernel_of<T, Ns + 1, P, VEC, false>() : k), ...);
    return k;
}
template <typename T, int P, bool VEC, int... Ns>
Kernel pick_wide(int order, std::integer_sequence<int, Ns...>) {
    Kernel k;
    ((k = (order == Ns + kWideFrom) ? kernel_of<T, Ns + kWideFrom, P, VEC, true>() : k), ...);
    return k;
}
template <typename T, int P, bool VEC, int MAX>
Kernel pick(int order, bool wide) {
    return wide ? pick_wide<T, P, VEC>(order, std::make_integer_sequence<int, kWideTo - kWideFrom + 1>{})
                : pick<T, P, VEC>(order, std::make_integer_sequence<int, MAX>{});
}

}  // namespace lattice_detail

int lattice_max_order(int dtype) { return dtype == 1 ? kLatticeMaxOrderC128 : kLatticeMaxOrderC64; }

hipError_t launch_lattice_step(const LatticeArgs& a, int dtype, int order, int cols, bool vec, bool wide, hipStream_t s) {
    using namespace lattice_detail;
    const Kernel k = dtype == 1 ? pick<double, 1, false, kLatticeMaxOrderC128>(order, wide)
                     : cols == 1 ? pick<float, 1, false, kLatticeMaxOrderC64>(order, wide)
                     : vec       ? pick<float, 2, true, kLatticePairOrder>(order, wide)
                                 : pick<float, 2, false, kLatticePairOrder>(order, wide);
    if (!k.fn || (dtype == 1 && cols != 1)) return hipErrorInvalidValue;
    if (k.lds > 64 * 1024) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(k.fn),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)k.lds);
        if (e != hipSuccess) return e;
    }
    const unsigned blocks = (unsigned)((a.n_items + 3) / 4);
    hipLaunchKernelGGL(k.fn, dim3(blocks), dim3(256), k.lds, s, a);
    return hipGetLastError();
}

hipError_t launch_lattice_norms(const double* part, int32_t per, int32_t R, int32_t steps, double* out, hipStream_t s) {
    const int64_t n = (int64_t)R * steps;
    hipLaunchKernelGGL(lattice_detail::lattice_norm_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, part,
                       per, R, steps, out);
    return hipGetLastError();
}

}  // namespace ctqw

// ------------------------------------------------------------------ C ABI

namespace {

using namespace ctqw;

int64_t align256(int64_t x) { return (x + 255) & ~int64_t(255); }

// The workspace: a second state, and as many bytes as three tables of the
// lattice and a partial per 64-column band hold.  That region takes the norm
// partials of up to kNormSteps steps, which wait for one reduction (bands and
// segments of a realisation are fewer than its nodes, so one step fits).
constexpr int kNormSteps = 8;

struct LatticeLayout {
    int64_t state = 0, part = 0, total = 0;
    int32_t cols = 1, nb = 0, segs = 1, held = 1;
};

ctqw_status lat_fail(ctqw_status st, const char* msg) { return (ctqw_status)report_error(st, msg); }

ctqw_status lattice_layout(int32_t Lx, int32_t Ly, int32_t R, int32_t dtype, int32_t order, int32_t periodic_x,
                           LatticeLayout* lay) {
    if (Lx < 1 || Ly < 1 || R < 1) return lat_fail(CTQW_ERR_INVALID_ARG, "need Lx, Ly, R >= 1");
    if (periodic_x && Lx < 3) return lat_fail(CTQW_ERR_INVALID_ARG, "a ring needs at least 3 nodes");
    if (dtype != CTQW_C64 && dtype != CTQW_C128) return lat_fail(CTQW_ERR_INVALID_ARG, "unknown dtype");
    const int maxo = lattice_max_order(dtype == CTQW_C128 ? 1 : 0);
    if (order < 1 || order > maxo) {
        char m[128];
        snprintf(m, sizeof m, "order must be in 1..%d for this dtype (got %d)", maxo, order);
        return lat_fail(order < 1 ? CTQW_ERR_INVALID_ARG : CTQW_ERR_UNSUPPORTED, m);
    }
    if ((int64_t)Lx * Ly * R > ((int64_t)1 << 31) / 3)
        return lat_fail(CTQW_ERR_UNSUPPORTED, "lattice tables beyond 2^31 entries");
    if ((int64_t)Lx * (dtype == CTQW_C128 ? 16 : 8) > ((int64_t)1 << 30))
        return lat_fail(CTQW_ERR_UNSUPPORTED, "rows beyond 2^30 bytes");
    using lattice_detail::band_count;
    using lattice_detail::halo_of;
    LatticeLayout l;
    l.nb = band_count(Lx, order, periodic_x != 0);
    if (l.nb <= 0) return lat_fail(CTQW_ERR_UNSUPPORTED, "order too deep for the band width");
    if ((int64_t)l.nb * R > INT32_MAX / 2) return lat_fail(CTQW_ERR_UNSUPPORTED, "too many work items");
    const int nb64 = l.nb;
    // One or two columns per lane (complex64, up to 10 terms: above, two spill)
    // and the rows of a band whole or in segments of at least `order` rows,
    // swept `order` rows early and late: the cheapest launch.  A sweep costs
    // its rows and the pipeline's depth in whole unrolled blocks, a row (10
    // terms, us, w waves on a SIMD) max(0.55, 0.38 w) with one complex64 column
    // per lane -- one wave alone waits more than it works --, 0.8 w with two,
    // and max(0.75, 0.52 w) in complex128.  (128 x 128, 1000 realisations, 10
    // terms: 127 us per step with two columns, 175 with one; 129 x 100, 500
    // realisations: 96 and 86; 300 x 300, one realisation: 30 us in segments,
    // 144 whole; 64 rings of 97 x 65, complex128, 9 terms: 30 and 51.)
    {
        constexpr int64_t kSimds = 1024;
        auto cost = [&](int64_t items, int64_t sg, int cols) {
            const int64_t steps = (Ly + sg - 1) / sg + (sg > 1 ? 2 * order : 0) + order;
            const int64_t w = (items * sg + kSimds - 1) / kSimds;
            const int64_t row = cols == 2 ? 32 * w : (dtype == CTQW_C64 ? std::max<int64_t>(22, 15 * w)
                                                                        : std::max<int64_t>(30, 21 * w));
            return lattice_detail::swept_rows(steps, order, false) * row;
        };
        int64_t best = INT64_MAX;
        for (int cols : {1, 2}) {
            if (cols == 2 && (dtype != CTQW_C64 || order > kLatticePairOrder)) break;
            const int nb = cols == 1 ? l.nb : band_count(Lx, halo_of(order, 2), periodic_x != 0, 128);
            const int64_t items = (int64_t)nb * R, most = items < kSimds ? std::max(1, Ly / order) : 1;
            for (int64_t sg = 1; sg <= most; ++sg) {
                const int64_t c = cost(items, sg, cols);
                if (c >= best) continue;
                best = c;
                l.cols = cols;
                l.segs = (int32_t)sg;
            }
        }
        if (l.cols == 2) l.nb = band_count(Lx, halo_of(order, 2), periodic_x != 0, 128);
    }
    const int64_t n = (int64_t)Lx * Ly * R;
    const int64_t csz = dtype == CTQW_C128 ? 16 : 8;
    l.state = 0;
    l.part = align256(l.state + n * csz);
    l.total = align256(align256(l.part + 3 * n * (csz / 2)) + (int64_t)nb64 * R * 8);
    const int64_t per = (int64_t)l.nb * l.segs * R * 8;
    l.held = (int32_t)std::min<int64_t>(kNormSteps, (l.total - l.part) / per);
    if (l.held < 1) return lat_fail(CTQW_ERR_UNSUPPORTED, "partials beyond the workspace");
    *lay = l;
    return CTQW_OK;
}

}  // namespace

extern "C" ctqw_status ctqw_lattice_workspace(int32_t Lx, int32_t Ly, int32_t R, int32_t dtype, int32_t order,
                                              int32_t periodic_x, int64_t* bytes) {
    if (!bytes) return lat_fail(CTQW_ERR_INVALID_ARG, "NULL argument");
    LatticeLayout l;
    const ctqw_status st = lattice_layout(Lx, Ly, R, dtype, order, periodic_x, &l);
    if (st != CTQW_OK) return st;
    *bytes = l.total;
    return CTQW_OK;
}

extern "C" ctqw_status ctqw_lattice_evolve(int32_t Lx, int32_t Ly, int32_t periodic_x, int32_t periodic_y, int32_t R,
                                           const void* Jx, const void* Jy, const void* eps, int32_t dtype, double dt,
                                           int32_t order, int64_t n_steps, void* psi, void* workspace,
                                           int64_t workspace_bytes, double* norms, void* hip_stream) {
    LatticeLayout l;
    ctqw_status st = lattice_layout(Lx, Ly, R, dtype, order, periodic_x, &l);
    if (st != CTQW_OK) return st;
    if (!Jx || !Jy || !eps || !psi || !workspace) return lat_fail(CTQW_ERR_INVALID_ARG, "NULL argument");
    if (periodic_y && Ly < 3) return lat_fail(CTQW_ERR_INVALID_ARG, "a ring needs at least 3 nodes");
    if (!std::isfinite(dt)) return lat_fail(CTQW_ERR_INVALID_ARG, "dt must be finite");
    if (n_steps < 0) return lat_fail(CTQW_ERR_INVALID_ARG, "n_steps must be >= 0");
    if (workspace_bytes < l.total) return lat_fail(CTQW_ERR_INVALID_ARG, "workspace too small");
    if (reinterpret_cast<uintptr_t>(workspace) & 255) return lat_fail(CTQW_ERR_INVALID_ARG, "workspace must be 256-byte aligned");
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    const int d = dtype == CTQW_C128 ? 1 : 0;
    char* ws = static_cast<char*>(workspace);
    auto hip_fail = [](hipError_t e) { return lat_fail(CTQW_ERR_DEVICE, hipGetErrorString(e)); };
    hipError_t e;
    LatticeArgs a{};
    a.Jx = Jx;
    a.Jy = Jy;
    a.eps = eps;
    a.Lx = Lx;
    a.Ly = Ly;
    a.R = R;
    a.px = periodic_x != 0;
    a.py = periodic_y != 0;
    a.nb = l.nb;
    a.segs = l.segs;
    a.n_items = l.nb * l.segs * R;
    a.dt = dt;
    // a lane's two columns in one access: even rows of aligned arrays
    const bool vec = l.cols == 2 && Lx % 2 == 0 &&
                     ((reinterpret_cast<uintptr_t>(psi) | reinterpret_cast<uintptr_t>(Jx) | reinterpret_cast<uintptr_t>(Jy) |
                       reinterpret_cast<uintptr_t>(eps)) & 15) == 0;
    // the rows of the longest sweep: output rows, the halo above and below (on an
    // open axis to its ends only) and the pipeline's depth
    const int out_rows = (Ly + l.segs - 1) / l.segs, halos = std::min(l.segs - 1, 2);
    const int64_t sweep = a.py ? out_rows + 2 * order : std::min(out_rows + halos * order, Ly);
    const bool wide = lattice_detail::wide_ring(sweep + order, order);
    double* const part = reinterpret_cast<double*>(ws + l.part);
    const int64_t bytes = (int64_t)Lx * Ly * R * (d ? 16 : 8);
    void* buf[2] = {psi, ws + l.state};
    int held = 0;   // steps whose partials are not reduced yet
    for (int64_t k = 0; k < n_steps; ++k) {
        a.psi_in = buf[k & 1];
        a.psi_out = buf[(k + 1) & 1];
        a.norm_part = part + (int64_t)held * a.n_items;
        if ((e = launch_lattice_step(a, d, order, l.cols, vec, wide, s)) != hipSuccess) return hip_fail(e);
        if (!norms) continue;
        ++held;
        if (held == l.held || k + 1 == n_steps) {
            if ((e = launch_lattice_norms(part, l.nb * l.segs, R, held, norms + (k + 1 - held) * (int64_t)R, s)) != hipSuccess)
                return hip_fail(e);
            held = 0;
        }
    }
    if (n_steps & 1) {
        e = (reinterpret_cast<uintptr_t>(psi) & 15) == 0
                ? launch_copy(psi, ws + l.state, bytes, s)
                : hipMemcpyAsync(psi, ws + l.state, bytes, hipMemcpyDeviceToDevice, s);
        if (e != hipSuccess) return hip_fail(e);
    }
    return CTQW_OK;
}
