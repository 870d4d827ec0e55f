// Device helpers shared by the kernel sources.
#pragma once
#include "bxmg_internal.h"

namespace bxmg {

// Raw-buffer resources (a base, a size in bytes, 32-bit lane offsets).
constexpr int kBufferDword3 = 0x00020000;  // raw buffer, gfx9 data format
// A lane offset beyond every box resource (their sizes stay below 2^31 bytes):
// the access is dropped.  The hardware compares it with the resource's size
// less the scalar offset, so that must not be negative: a plane below the box
// would take away what is left up to 2^31, and in the largest boxes the
// access would land in their last planes.
constexpr int kOffPastBox = (int)0x80000000u;

// a / b for a loop-invariant b whose reciprocal is held in two parts,
// 1/b = yh + yl: the estimate fma(a, yh, a yl) is within half an ulp and a
// rounding of a/b, and the correction by its exact remainder then gives the
// correctly rounded quotient (Markstein 1990) -- the IEEE division's bits,
// in 4 dependent instructions instead of about 12.  (An infinite a gives NaN;
// both end the solve as non-finite.)
template <class T>
struct Recip {
    T b, yh, yl;
    __device__ __forceinline__ explicit Recip(T d) : b(d), yh(T(1) / d), yl(fma_(-d, yh, T(1)) * yh) {}
    static __device__ __forceinline__ double fma_(double x, double y, double z) { return __builtin_fma(x, y, z); }
    static __device__ __forceinline__ float fma_(float x, float y, float z) { return __builtin_fmaf(x, y, z); }
    __device__ __forceinline__ T div(T a) const {
        const T q = fma_(a, yh, a * yl);
        return fma_(fma_(-q, b, a), yh, q);
    }
};

// Barrier between LDS writers and readers of one step; global loads in
// flight (the planes ahead) and stores are not waited for.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

template <class T>
struct Raw;
template <>
struct Raw<double> {
    static __device__ __forceinline__ double ld(__amdgpu_buffer_rsrc_t r, int v, int s) {
        return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, v, s, 0));
    }
    static __device__ __forceinline__ void st(__amdgpu_buffer_rsrc_t r, int v, int s, double x) {
        typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, x), r, v, s, 0);
    }
};
template <>
struct Raw<float> {
    static __device__ __forceinline__ float ld(__amdgpu_buffer_rsrc_t r, int v, int s) {
        return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, v, s, 0));
    }
    static __device__ __forceinline__ void st(__amdgpu_buffer_rsrc_t r, int v, int s, float x) {
        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned int, x), r, v, s, 0);
    }
};

template <class T>
__device__ __forceinline__ T harm(T a, T b) {
    return (a * b) * T(2) / (a + b);
}

// A value that is the same in every lane, into scalar registers.
__device__ __forceinline__ float uniform(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, v)));
}
__device__ __forceinline__ double uniform(double v) {
    const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
    const unsigned lo = __builtin_amdgcn_readfirstlane((int)(unsigned)b);
    const unsigned hi = __builtin_amdgcn_readfirstlane((int)(unsigned)(b >> 32));
    return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}

// Fixed-tree block reduction of (max, sum, sum): wave64 butterflies, then
// the 4 wave results in order.  The result is valid in thread 0.
__device__ __forceinline__ void block_reduce3(double& mx, double& s2, double& bad, double* sh) {
    for (int o = 32; o > 0; o >>= 1) {
        const double a = __shfl_xor(mx, o), b = __shfl_xor(s2, o), c = __shfl_xor(bad, o);
        mx = fmax(mx, a);
        s2 = s2 + b;
        bad = bad + c;
    }
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    if (lane == 0) { sh[3 * wid] = mx; sh[3 * wid + 1] = s2; sh[3 * wid + 2] = bad; }
    __syncthreads();
    if (threadIdx.x == 0) {
        const int nw = (blockDim.x + 63) >> 6;
        mx = sh[0]; s2 = sh[1]; bad = sh[2];
        for (int w = 1; w < nw; ++w) { mx = fmax(mx, sh[3 * w]); s2 = s2 + sh[3 * w + 1]; bad = bad + sh[3 * w + 2]; }
    }
}

// Sums kept as s + c, c the rounding errors of s and of the products (Ogita,
// Rump and Oishi 2005): as if summed in twice the precision, so that a sum
// does not depend on how its terms are split over threads and blocks.  (An
// infinite s makes c NaN: sum2 drops it.)
struct Sum2 {
    double s = 0.0, c = 0.0;
    __device__ __forceinline__ void add(double x, double e) {
        const double t = s + x, z = t - s;
        c = c + (((s - (t - z)) + (x - z)) + e);
        s = t;
    }
    __device__ __forceinline__ void dot(double a, double b) {
        const double x = a * b;
        add(x, __builtin_fma(a, b, -x));
    }
    __device__ __forceinline__ double value() const { return fabs(s) <= 1.7976931348623157e308 ? s + c : s; }
};

// Fixed-tree block sum of v; the result is valid in thread 0 (sh: 2 per wave).
__device__ __forceinline__ void block_sum2(Sum2& v, double* sh) {
    for (int o = 32; o > 0; o >>= 1) {
        const double x = __shfl_xor(v.s, o), e = __shfl_xor(v.c, o);
        v.add(x, e);
    }
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    __syncthreads();
    if (lane == 0) { sh[2 * wid] = v.s; sh[2 * wid + 1] = v.c; }
    __syncthreads();
    if (threadIdx.x == 0) {
        const int nw = (blockDim.x + 63) >> 6;
        v.s = sh[0];
        v.c = sh[1];
        for (int w = 1; w < nw; ++w) v.add(sh[2 * w], sh[2 * w + 1]);
    }
}

// A block's partial sums of two dots (launch_kr_sums).
__device__ __forceinline__ void store_sums(double* __restrict__ partials, int blk, const Sum2& a, const Sum2& b) {
    double* o = partials + 4 * (size_t)blk;
    o[0] = a.s;
    o[1] = a.c;
    o[2] = b.s;
    o[3] = b.c;
}

__device__ __forceinline__ void acc_norm(double rv, double& mx, double& s2, double& bad) {
    const double a = fabs(rv);
    if (!(a <= 1.7976931348623157e308)) bad += 1.0;  // NaN or Inf
    else mx = fmax(mx, a);
    s2 = s2 + rv * rv;
}

}  // namespace bxmg
