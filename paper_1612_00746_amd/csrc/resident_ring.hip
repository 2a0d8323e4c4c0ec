// Resident kernels: full grids on rings.
#include "resident_impl.hpp"

namespace ctqw {
namespace {
template <typename T, bool KAHAN>
ResidentFn pick(const ResidentShape& s) {
    constexpr int LAYOUT = kResRing;
    CTQW_RESIDENT(1, 2, 1024)
    CTQW_RESIDENT(1, 4, 1024)
    CTQW_RESIDENT(1, 8, 512)
    if constexpr (sizeof(T) == 8) {
        CTQW_RESIDENT(2, 10, 512)
        CTQW_RESIDENT(2, 12, 512)
    }
    return {};
}
}  // namespace

ResidentFn resident_ring(const ResidentShape& s) {
    if (s.dtype) return pick<double, false>(s);
    return s.kahan ? pick<float, true>(s) : pick<float, false>(s);
}
}  // namespace ctqw
