// 16-byte vector access along the channels and the batch-norm coefficients of a channel: shared by the HBM-bound passes
// and by the convolution kernels that apply a batch norm to what they load.
#pragma once
#include "lp_kernels.h"
#include "lp_mma.h"

namespace lp {

template <typename T> struct Vec {
    static constexpr int N = 16 / (int)sizeof(T);
    __device__ static __forceinline__ void load(const T* p, float (&f)[N]) {
        const u32x4 v = *reinterpret_cast<const u32x4*>(p);
        if constexpr (sizeof(T) == 4) {
#pragma unroll
            for (int e = 0; e < 4; ++e) f[e] = __uint_as_float(v[e]);
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                f[2 * e] = __uint_as_float(v[e] << 16);
                f[2 * e + 1] = __uint_as_float(v[e] & 0xffff0000u);
            }
        }
    }
    // the 16 bytes as loaded, and their conversion: kernels that want many loads in flight issue all load_raw first
    __device__ static __forceinline__ u32x4 load_raw(const T* p) { return *reinterpret_cast<const u32x4*>(p); }
    __device__ static __forceinline__ void unpack(const u32x4& v, float (&f)[N]) {
        if constexpr (sizeof(T) == 4) {
#pragma unroll
            for (int e = 0; e < 4; ++e) f[e] = __uint_as_float(v[e]);
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                f[2 * e] = __uint_as_float(v[e] << 16);
                f[2 * e + 1] = __uint_as_float(v[e] & 0xffff0000u);
            }
        }
    }
    __device__ static __forceinline__ u32x4 pack(const float (&f)[N]) {
        u32x4 v;
        if constexpr (sizeof(T) == 4) {
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = __float_as_uint(f[e]);
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                v[e] = pack_bf16x2(f[2 * e], f[2 * e + 1]);
        }
        return v;
    }
    __device__ static __forceinline__ void store(T* p, const float (&f)[N]) { *reinterpret_cast<u32x4*>(p) = pack(f); }
};

// the two per-channel sums of channel c, their stripes added in order; all loads of up to eight stripes are under way at
// once (behind a loop of unknown length they would be requested one after the other)
__device__ __forceinline__ void stripe_sums(const double* p, int c, int C, double& s1, double& s2) {
    const int ns = stat_stripes(C);
    double a[kStatStripes], b[kStatStripes];
    if (ns == kStatStripes) {
#pragma unroll
        for (int st = 0; st < kStatStripes; ++st) { a[st] = p[st * 2 * C + c]; b[st] = p[st * 2 * C + C + c]; }
        s1 = a[0]; s2 = b[0];
#pragma unroll
        for (int st = 1; st < kStatStripes; ++st) { s1 += a[st]; s2 += b[st]; }
        return;
    }
    s1 = 0.0; s2 = 0.0;
    for (int st = 0; st < ns; ++st) { s1 += p[st * 2 * C + c]; s2 += p[st * 2 * C + C + c]; }
}
// the same in two parts, for loads that are to be under way before they are waited for
struct StripeLoads {
    double a[kStatStripes], b[kStatStripes];
    int ns;
    __device__ __forceinline__ void load(const double* p, int c, int C) {
        ns = stat_stripes(C);
#pragma unroll
        for (int st = 0; st < kStatStripes; ++st) {
            const int o = (st < ns ? st : 0) * 2 * C + c;
            a[st] = p[o]; b[st] = p[o + C];
        }
    }
    __device__ __forceinline__ void sums(double& s1, double& s2) const {
        s1 = a[0]; s2 = b[0];
#pragma unroll
        for (int st = 1; st < kStatStripes; ++st)
            if (st < ns) { s1 += a[st]; s2 += b[st]; }
    }
};
__device__ __forceinline__ void bn_coeffs(const StripeLoads& l, float gamma, float beta, int M, float eps, float& sc, float& sh, float& mean, float& invstd) {
    const double inv_m = 1.0 / (double)M;
    double s1, s2;
    l.sums(s1, s2);
    const double mu = s1 * inv_m;
    double var = s2 * inv_m - mu * mu;
    if (var < 0.0) var = 0.0;
    mean = (float)mu;
    invstd = rsqrtf((float)var + eps);
    sc = gamma * invstd;
    sh = beta - mean * sc;
}
__device__ __forceinline__ void bn_coeffs(const double* stats, const float* gamma, const float* beta, int c, int C,
                                          int M, float eps, float& sc, float& sh, float& mean, float& invstd) {
    const double inv_m = 1.0 / (double)M;          // the same for every channel: the compiler hoists it out of loops
    double s1, s2;
    stripe_sums(stats, c, C, s1, s2);
    const double mu = s1 * inv_m;
    double var = s2 * inv_m - mu * mu;
    if (var < 0.0) var = 0.0;
    mean = (float)mu;
    invstd = rsqrtf((float)var + eps);
    sc = gamma[c] * invstd;
    sh = beta[c] - mean * sc;
}

}  // namespace lp
