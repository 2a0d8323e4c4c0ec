// Steps of small lattices with the state held on chip (resident.hip).
#pragma once

#include "ctqw_internal.hpp"

#include <vector>

namespace ctqw {

// Deepest series of the resident kernel (its coefficients are arguments).
constexpr int kResidentMaxOrder = 64;

// Grid of one realisation as the resident kernel holds it.
enum : int { kResFull = 0, kResRing = 1, kResTri = 2 };

struct ResidentArgs {
    const void* psi_in;
    void* psi_out;           // may be psi_in: a block reads its whole realisation first
    int64_t out_stride;      // bytes; > 0: the state after step s is stored at psi_out + s * out_stride,
                             // 0: the last state alone
    const RealDev* reals;
    const void* Jt;          // dt-scaled tables (dtype of the state)
    const void* Et;
    double* scale;           // [R] load scale, in and out
    double* norm2;           // [R] after the last step; null: no monitoring
    double* tail2;
    int32_t* status;
    int64_t steps;
    double dt;
    double tol2;             // as FinalizeArgs
    double norm_alarm;
    int32_t renormalize;
    int32_t one_order;       // > 0: every realisation at this order (the batch's largest)
    double coef[kResidentMaxOrder + 4];   // 1/j! (read up to two terms ahead)
};

struct ResidentShape {
    int layout;     // kRes*
    int dtype;      // 0: complex64, 1: complex128
    int kahan;
    int cols;       // columns per lane
    int rows;       // rows per wave
    int waves;      // waves per block
    int max_N;      // largest lattice of the batch
};

// Shape for the batch's largest lattice, or false if a realisation's state
// does not fit one compute unit (or the order is too deep).
bool resident_shape(int layout, int dtype, int kahan, int max_N, int max_order, int64_t R, ResidentShape* out);
// One step of the batch as band sweeps.
struct BandLaunch {
    int order = 0;          // terms
    int64_t items = 0;
    int64_t rows = 0;       // swept, over all items, with the pipeline's depth
    int longest = 0;        // of one item
};
// Estimated us of a step in these launches (passes > 1: the one launch is each
// pass's share).
double band_step_us(int layout, int dtype, int cols, int passes, const std::vector<BandLaunch>& launches, int64_t bytes);
// Whether `steps` steps (of `bytes` of state, each band_us as bands) take less
// time on chip.
bool resident_pays(const ResidentShape& s, int64_t R, int order, int64_t bytes, int64_t steps, double band_us);
// A compiled shape: its kernel, the block it was compiled for, its LDS bytes.
struct ResidentFn {
    void (*kernel)(ResidentArgs) = nullptr;
    int max_threads = 0;
    size_t (*lds)(const ResidentShape&) = nullptr;
};
ResidentFn resident_full(const ResidentShape& s);
ResidentFn resident_ring(const ResidentShape& s);
ResidentFn resident_tri(const ResidentShape& s);
hipError_t launch_resident(const ResidentShape& s, const ResidentArgs& a, int64_t R, hipStream_t stream);

}  // namespace ctqw
