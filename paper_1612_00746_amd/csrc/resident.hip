// Choice and launch of the resident kernel (resident_impl.hpp; instantiated
// in resident_full.hip, resident_ring.hip and resident_tri.hip).
#include "resident.hpp"

namespace ctqw {
namespace {

constexpr size_t kLdsBytes = 160 * 1024;   // of one compute unit

ResidentFn kernel_of(const ResidentShape& s) {
    if (s.layout == kResTri) return resident_tri(s);
    return s.layout == kResRing ? resident_ring(s) : resident_full(s);
}

}  // namespace

// Which batches run on chip, and in which shape.  A realisation's vector and
// sums (complex64: and its state) have to fit the 2048 registers x 64 lanes
// of a compute unit with room to work in: 128 columns (two per lane), except
// complex128 full grids, where 96 rows is the last size that does not spill
// heavily.  Times per step against the swept bands of step2d_impl.hpp, 1000
// realisations (orders 12 complex128, 7 complex64):
//   bosons  N = 128: 90 / 733 us, complex64 43 / 135;  N = 64: 27 / 250, 12 / 46
//   grid    N = 96: 127 / 284, complex64 41 / 59;  N = 64: 43 / 147, 16 / 33
//   16 realisations, bosons N = 64: 9 / 153, complex64 5 / 29
// A complex64 ring wider than 64 columns gains nothing (67 / 63 at N = 96:
// the lanes that close the ring cost more than the bands' halos), so it
// stays on the bands.
//
// Rows per wave: with no more realisations than compute units a step lasts
// as long as one block's levels, so few rows per wave (more waves at work);
// above, blocks share compute units and the exchange of edge rows is what
// costs, so more rows per wave.  Measured, us per step at N = 32, order 7:
// 16 bosonic realisations 3.9 / 4.3 / 4.8 / 6.6 for 2 / 3 / 5 / 9 rows, 1000
// realisations 12.2 / 8.8 / 7.5 / 7.7.
bool resident_shape(int layout, int dtype, int kahan, int max_N, int max_order, int64_t R, ResidentShape* out) {
    if (max_order > kResidentMaxOrder || max_N > 128) return false;
    constexpr int64_t kComputeUnits = 256;
    const bool tri = layout == kResTri, few = R <= kComputeUnits;
    const int K = tri ? max_N / 2 + 1 : max_N;   // rows held
    ResidentShape s{};
    s.layout = layout;
    s.dtype = dtype;
    s.kahan = dtype ? 0 : kahan;
    s.cols = max_N <= 64 ? 1 : 2;
    s.max_N = max_N;
    if (s.cols == 1) {
        if (tri) s.rows = few ? (K <= 32 ? 2 : 3) : (K <= 9 ? 3 : (K <= 17 ? 5 : 9));
        else s.rows = few ? (K <= 32 ? 2 : 4) : (K <= 16 ? 4 : 8);
    } else if (tri) {
        s.rows = dtype ? 9 : 5;
    } else if (dtype) {
        if (K > 96) return false;
        s.rows = K <= 80 ? 10 : 12;
    } else {
        if (layout == kResRing) return false;
        s.rows = K <= 96 ? 6 : 16;
    }
    s.waves = (K + s.rows - 1) / s.rows;
    const ResidentFn fn = kernel_of(s);
    if (!fn.kernel || 64 * s.waves > fn.max_threads || fn.lds(s) > kLdsBytes) return false;
    *out = s;
    return true;
}

hipError_t launch_resident(const ResidentShape& s, const ResidentArgs& a, int64_t R, hipStream_t stream) {
    const ResidentFn fn = kernel_of(s);
    // a launch takes fewer than 2^32 threads along x
    if (!fn.kernel || R < 1 || R * 64 * s.waves > UINT32_MAX || 64 * s.waves > fn.max_threads)
        return hipErrorInvalidValue;
    const size_t lds = fn.lds(s);
    if (lds > kLdsBytes) return hipErrorInvalidValue;
    if (lds > 64 * 1024) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(fn.kernel),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(fn.kernel, dim3((unsigned)R), dim3(64 * s.waves), lds, stream, a);
    return hipGetLastError();
}

}  // namespace ctqw
