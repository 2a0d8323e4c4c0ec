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
// heavily.  Which calls of such a batch run on chip is resident_pays' choice.
// Times per step against the swept bands of step2d_impl.hpp, 1000 realisations
// (orders 12 complex128, 7 complex64):
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

// On chip every block does the work of the shape, that is of the batch's
// largest lattice, and moves its state between launches with nothing to
// overlap it; a band sweep does each realisation's own work and overlaps the
// traffic, but moves the state once per step.  So the bands win where most
// realisations are much smaller than the largest, and, for states that pass
// the last-level cache, where a call takes few steps.  us on chip / as bands:
//   complex64 grid, 4095 of 16 nodes and one of 128, 20 steps: 4330 / 1290
//   complex64 grid N = 96, R = 8000: 1 step 639 / 362, 16 steps 5286 / 5628
//   complex64 ring N = 48, R = 16000, 16 steps: 5730 / 3760
//   complex64 grid N = 64, R = 1000, 30 steps: 452 / 1505
// The two estimates' constants are fits to 1500 random batches (1 to 65535
// realisations of 3 to 128 nodes, equal and mixed, 2 to 20 terms, calls of 1,
// 2, 4 and 16 steps), 12 and 15 % rms: under 1 % of the calls take the chip and
// 1.3 % the bands where the other is more than 4 % faster, on average 0.3 %;
// always on chip, 10 (16 steps) to 19 % (one) did, up to fourfold.  complex64
// grids give the same bits either way; the other states agree to rounding.
double band_step_us(int layout, int dtype, int cols, int passes, const std::vector<BandLaunch>& launches, int64_t bytes) {
    const bool tri = layout == kResTri, f64 = dtype != 0, chunked = passes > 1;
    constexpr double kSimds = 1024, kStart = 6;   // rows' time that an item's start takes
    // us per row and level: of a SIMD with work to spare, and of one sweep alone
    double row = f64 ? 0.053 : (tri ? 0.037 : 0.029);
    double alone = f64 ? (tri ? 0.097 : 0.069) : (tri ? 0.057 : 0.044);
    if (cols == 2) {
        row *= tri ? 2.55 : 1.75;
        alone *= tri ? 3.0 : 1.7;
    }
    if (chunked) {
        row *= f64 ? 1.2 : 1.4;
        alone *= f64 ? 1.2 : 1.4;
    }
    // from some order on a kernel holds one wave per SIMD instead of two
    const int one_wave = (f64 ? (tri ? 6 : 8) : (tri ? 10 : 12)) - (cols == 2 ? 3 : 0);
    const double lone = f64 ? (tri ? 2.0 : 1.4) : (tri ? 1.5 : 1.6);
    double us = 2.0;
    for (const BandLaunch& l : launches) {
        const double r = !chunked && l.order >= one_wave ? row * lone : row;
        us += std::max(alone * l.longest * l.order, r * ((double)l.rows + kStart * (double)l.items) * l.order / kSimds);
    }
    us += 5.5 * (chunked ? passes : (double)launches.size());
    // (a chunked pass reads and writes the sum and the last term)
    return std::max(us, (chunked ? 4.0 * passes : 2.0) * (double)bytes / 3.7e6);
}

bool resident_pays(const ResidentShape& s, int64_t R, int order, int64_t bytes, int64_t steps, double band_us) {
    const bool tri = s.layout == kResTri, ring = s.layout == kResRing, f64 = s.dtype != 0;
    constexpr double kComputeUnits = 256;
    // One level: a wave's issue per row and column (closing the ring costs more,
    // and FP64 rows that spill), times the waves that a compute unit holds;
    // fewer, larger blocks wait as long for each other.
    const int held = f64 ? (s.rows <= 5 ? 16 : 8) : (s.rows == 16 ? 8 : 16);
    const int blocks = std::max(1, held / s.waves);
    double issue = f64 ? (tri ? 11.7e-3 : (ring ? 19e-3 : 9.7e-3)) : (tri ? 7.7e-3 : (ring ? 12.8e-3 : 7.1e-3));
    if (f64 && !tri && blocks == 1 && (s.rows == 8 || s.rows == 12)) issue *= 1.33;
    const double full = issue * held * s.rows * s.cols;
    const double level = std::max(0.11 + 0.85 * full, full / blocks * (double)R / kComputeUnits);
    // the state read and written (two columns of a triangle per lane lie scattered)
    const double spread = s.cols == 1 ? 1.0 : (tri ? 2.0 : 1.17);
    const double start = s.cols == 1 ? 0.5 : (s.rows >= 12 ? 8.0 : 3.0);
    const double on_chip = start + 2.0 * (double)bytes * spread / 4.85e6 +
                           (double)steps * (order + 1) * level;
    return on_chip < (double)steps * band_us;
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
