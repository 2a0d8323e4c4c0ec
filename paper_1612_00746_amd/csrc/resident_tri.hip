// Resident kernels: triangles of two bosons or fermions.
#include "resident_impl.hpp"

namespace ctqw {
namespace {
template <typename T, bool KAHAN>
ResidentFn pick(const ResidentShape& s) {
    constexpr int LAYOUT = kResTri;
    CTQW_RESIDENT(1, 2, 1024)
    CTQW_RESIDENT(1, 3, 1024)
    CTQW_RESIDENT(1, 5, 512)
    CTQW_RESIDENT(1, 9, 256)
    if constexpr (sizeof(T) == 4) {
        CTQW_RESIDENT(2, 5, 1024)
    } else {
        CTQW_RESIDENT(2, 9, 512)
    }
    return {};
}
}  // namespace

ResidentFn resident_tri(const ResidentShape& s) {
    if (s.dtype) return pick<double, false>(s);
    return s.kahan ? pick<float, true>(s) : pick<float, false>(s);
}
}  // namespace ctqw
