// Auxiliary kernels: start state, per-step FP64 norm / truncation check,
// rescaling.
#include "ctqw_internal.hpp"

namespace ctqw {
namespace {

__device__ __forceinline__ int64_t tri_index(int q, int c, int N) {
    return (int64_t)q * N - ((int64_t)q * (q + 1)) / 2 + c;
}

// ---------------------------------------------------------------- fill / init

__global__ void fill_zero_kernel(uint32_t* __restrict__ p, int64_t words) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (; i < words; i += stride) p[i] = 0u;
}

// One 16-byte element per thread, stored non-temporal (NT) or to the caches;
// the last thread also takes the bytes past the last whole element.
typedef float f32x4 __attribute__((ext_vector_type(4)));
template <bool NT>
__global__ __launch_bounds__(256) void copy_kernel(const f32x4* __restrict__ src, f32x4* __restrict__ dst, int64_t n,
                                                   int tail_words) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) {
        if (NT) __builtin_nontemporal_store(src[i], dst + i);
        else dst[i] = src[i];
    } else if (i == n)
        for (int k = 0; k < tail_words; ++k)
            reinterpret_cast<float*>(dst + n)[k] = reinterpret_cast<const float*>(src + n)[k];
}

template <typename C>
__global__ void init_sites_kernel(InitArgs a) {
    const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= a.R) return;
    const RealDev rd = a.reals[r];
    const int32_t* s = a.sites + (a.per_real ? r * a.m : 0);
    C* psi = reinterpret_cast<C*>(a.psi) + rd.state_off;
    C one;
    one.x = 1;
    one.y = 0;
    if (a.m == 1) {
        psi[s[0]] = one;
        return;
    }
    if (a.m == 3) {
        psi[((int64_t)s[0] * rd.N + s[1]) * rd.N + s[2]] = one;
        return;
    }
    int x1 = s[0], x2 = s[1];
    if (rd.flags & RF_TRIANGLE) {
        // bosons: phi(x1, x2) = phi(x2, x1) = 1/sqrt 2 (1 on the diagonal);
        // fermions: phi(x1, x2) = -phi(x2, x1) = 1/sqrt 2 for particle 1 on x1
        const bool swapped = x1 > x2;
        if (swapped) { const int t = x1; x1 = x2; x2 = t; }
        C v;
        v.x = (x1 == x2) ? 1.0 : 0.70710678118654752440;
        if ((rd.flags & RF_FERMION) && swapped) v.x = -v.x;
        v.y = 0;
        psi[tri_index(x1, x2, rd.N)] = v;
    } else {
        psi[(int64_t)x1 * rd.N + x2] = one;
    }
}

// ------------------------------------------------------------ step finalize

// One wave per realisation: lane l sums the partials l, l + 64, ... of its
// realisation, then a fixed butterfly combines the lanes (deterministic;
// three walkers have 65536 partials per realisation at N = 256).
__global__ void finalize_kernel(FinalizeArgs a) {
    const int64_t r = (int64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (r >= a.R) return;   // wave-uniform
    double s = 0.0, t = 0.0, err2 = 0.0;
    const int32_t k0 = a.item_first[r], k1 = a.item_first[r + 1];
    const double tf = a.use_max ? a.reals[r].tail_factor_max : a.reals[r].tail_factor;
    int flags = 0, alarms = 0;
    for (int m = 0; m < a.slots; ++m) {
        s = t = 0.0;
        for (int32_t k = k0 + lane; k < k1; k += 64) {
            s += a.norm_part[m * a.slot_stride + k];
            t += a.tail_part[m * a.slot_stride + k];
        }
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) {
            s += __shfl_xor(s, off, 64);
            t += __shfl_xor(t, off, 64);
        }
        err2 = t * tf * tf;
        int flag = 0;
        if (a.tol2 > 0.0 && !(err2 <= a.tol2 * s)) flag |= 1;
        if (!isfinite(s) || !isfinite(t)) flag |= 2;
        if (a.norm_alarm > 0.0 && !(fabs(sqrt(s) - 1.0) <= a.norm_alarm)) flag |= 2;
        flags |= flag;
        alarms += flag ? 1 : 0;
    }
    if (lane != 0) return;
    a.norm2[r] = s;
    a.tail2[r] = err2;
    if (flags) {
        atomicOr(&a.status[0], flags);
        atomicAdd(&a.status[1], alarms);
    }
    if (a.renormalize && s > 0.0 && isfinite(s)) a.scale[r] = 1.0 / sqrt(s);
}

// ------------------------------------------------------------------ rescale

template <typename C>
__global__ void rescale_kernel(RescaleArgs a) {
    const int64_t r = blockIdx.y;
    const RealDev rd = a.reals[r];
    const int64_t n = (rd.flags & RF_TRIANGLE) ? (int64_t)rd.N * (rd.N + 1) / 2 : (int64_t)rd.rows * rd.N;
    const double s = a.scale[r];
    C* psi = reinterpret_cast<C*>(a.psi) + rd.state_off;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        C v = psi[i];
        v.x = v.x * s;
        v.y = v.y * s;
        psi[i] = v;
    }
}

__global__ void reset_scale_kernel(double* scale, int64_t R) {
    const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (r < R) scale[r] = 1.0;
}

}  // namespace

hipError_t launch_fill_zero(void* p, int64_t bytes, hipStream_t stream) {
    if (bytes <= 0) return hipSuccess;
    if (bytes % 4) return hipErrorInvalidValue;
    const int64_t words = bytes / 4;
    int64_t blocks = (words + 255) / 256;
    if (blocks > 65536) blocks = 65536;
    hipLaunchKernelGGL(fill_zero_kernel, dim3((unsigned)blocks), dim3(256), 0, stream,
                       static_cast<uint32_t*>(p), words);
    return hipGetLastError();
}

// Device-to-device copy of whole states.  The runtime's copy moves a large
// state at 4.8 TB/s (read and written), this one at 6.2; it needs 16-byte
// aligned buffers of this device, whole 4-byte words, that do not overlap.
// Copies that fit the last-level cache (256 MB) are stored to it, as the
// runtime's are: back and forth, us per copy non-temporal / to the cache /
// runtime: 32 MB 14.0 / 11.6 / 11.5, 128 MB 42.5 / 38.4 / 38.4, 256 MB 85.9 /
// 82.5 / 99.5, 512 MB 169.5 / 168.4 / 200, 1 GB 335 / 344 / 411.
hipError_t launch_copy(void* dst, const void* src, int64_t bytes, hipStream_t stream) {
    if (bytes <= 0) return hipSuccess;
    if (bytes % 4 || ((reinterpret_cast<uintptr_t>(dst) | reinterpret_cast<uintptr_t>(src)) & 15))
        return hipErrorInvalidValue;
    const int64_t n = bytes / 16;
    const f32x4* from = static_cast<const f32x4*>(src);
    f32x4* to = static_cast<f32x4*>(dst);
    // a launch takes fewer than 2^32 threads along x: pieces of 16 GiB
    constexpr int64_t kPiece = int64_t(1) << 30;
    constexpr int64_t kCached = int64_t(256) << 20;
    const auto kernel = bytes <= kCached ? copy_kernel<false> : copy_kernel<true>;
    for (int64_t i = 0;; i += kPiece) {
        const int64_t m = std::min(n - i, kPiece);
        const bool last = i + m == n;
        hipLaunchKernelGGL(kernel, dim3((unsigned)(m / 256 + 1)), dim3(256), 0, stream, from + i, to + i, m,
                           last ? (int)(bytes % 16) / 4 : 0);
        if (last) return hipGetLastError();
    }
}

hipError_t launch_init(const InitArgs& a, hipStream_t stream) {
    const int64_t bytes = a.total * (a.dtype == 1 ? 16 : 8);
    hipError_t e = launch_fill_zero(a.psi, bytes, stream);
    if (e != hipSuccess) return e;
    const unsigned blocks = (unsigned)((a.R + 255) / 256);
    if (a.dtype == 1) hipLaunchKernelGGL(init_sites_kernel<double2>, dim3(blocks), dim3(256), 0, stream, a);
    else hipLaunchKernelGGL(init_sites_kernel<float2>, dim3(blocks), dim3(256), 0, stream, a);
    return hipGetLastError();
}

hipError_t launch_finalize(const FinalizeArgs& a, hipStream_t stream) {
    const unsigned blocks = (unsigned)((a.R + 3) / 4);   // four waves (realisations) per block
    hipLaunchKernelGGL(finalize_kernel, dim3(blocks), dim3(256), 0, stream, a);
    return hipGetLastError();
}

hipError_t launch_rescale(const RescaleArgs& a, hipStream_t stream) {
    if (a.R > 65535) return hipErrorInvalidValue;
    const dim3 g(64, (unsigned)a.R);
    if (a.dtype == 1) hipLaunchKernelGGL(rescale_kernel<double2>, g, dim3(256), 0, stream, a);
    else hipLaunchKernelGGL(rescale_kernel<float2>, g, dim3(256), 0, stream, a);
    hipLaunchKernelGGL(reset_scale_kernel, dim3((unsigned)((a.R + 255) / 256)), dim3(256), 0, stream, a.scale, a.R);
    return hipGetLastError();
}

}  // namespace ctqw
