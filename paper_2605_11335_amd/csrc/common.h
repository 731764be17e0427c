// Shared device-side types for the block kernels (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

typedef __bf16 bf16;
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef unsigned int uint32x2 __attribute__((ext_vector_type(2)));
typedef unsigned int uint32x4 __attribute__((ext_vector_type(4)));

// A block's weight blob as the kernels see it: bytes [0, split) of the blob live in the
// block's resident buffer (`lo`), bytes [split, blob) in the staging slot the prefetch fills
// (`hi`); both pointers are biased so that `ptr + blob_offset` addresses the byte.  `split`
// is a multiple of 256, so an aligned 16-byte access never straddles the two.
struct WView {
    const char* lo;
    const char* hi;
    uint64_t split;
};

__device__ __forceinline__ const char* wv_ptr(const WView& w, uint64_t boff) {
    return (boff < w.split ? w.lo : w.hi) + boff;
}

__device__ __forceinline__ float bf16_bits_to_float(uint16_t b) {
    return __uint_as_float(((uint32_t)b) << 16);
}

__device__ __forceinline__ float wv_bf16(const WView& w, uint64_t boff_of_tensor, uint32_t idx) {
    return bf16_bits_to_float(*(const uint16_t*)wv_ptr(w, boff_of_tensor + 2ull * idx));
}

// Workgroup id -> logical tile id such that each XCD (workgroups are dealt round-robin to the
// 8 XCDs) walks one contiguous range of logical ids and so shares operands in its own L2.
__host__ __device__ __forceinline__ uint32_t xcd_contiguous_id(uint32_t bid, uint32_t nb) {
    const uint32_t q = nb >> 3, r = nb & 7u;
    const uint32_t xcd = bid & 7u, idx = bid >> 3;
    return xcd < r ? xcd * (q + 1) + idx : r * (q + 1) + (xcd - r) * q + idx;
}

// x * sigmoid(2u), u = sqrt(2/pi) (x + 0.044715 x^3): the tanh form of GELU.  exp(-2u) = exp2(x (a + b x^2)) with the factors
// folded into a and b (an epilogue of 256 x 256 tiles evaluates it 256 times per lane: 1 % of 2304 x 21504 x 3072).
__device__ __forceinline__ float gelu_tanh_f32(float x) {
    const float en = __builtin_amdgcn_exp2f(x * fmaf(x * x, -0.1029432407f, -2.302208198f));
    return x * __builtin_amdgcn_rcpf(1.0f + en);
}

// x * Phi(x), the GELU the tanh form approximates, by the rational-times-Gaussian formula of Abramowitz & Stegun 7.1.26 for
// erfc (absolute error below 1.5e-7, far under a bf16 ulp of a result of ordinary size):
// erfc(z) = (a1 t + ... + a5 t^5) exp(-z^2), t = 1 / (1 + p z), z = |x| / sqrt 2 >= 0, and x Phi(x) = max(x, 0) - 0.5 |x| erfc(z):
// nothing cancels in the negative tail, where the formula's relative error is what is left (0.4 % of the result at x = -6, 1 % at
// -8, 3 % at -12: results of 6e-9, 5e-15 and 2e-32).  The factor |x| is held to 20, from where on erfc(z) is zero in fp32: an
// infinite one would make +inf a NaN; a NaN still comes through erfc.  Seventeen operations with the hardware's reciprocal and
// exponential (1 ulp each); with a correctly rounded reciprocal and exp2f it was some sixty, 8 us more per generation of
// 256 x 256 tiles (1320 x 14336 x 3072: 166 -> 150 us).
__device__ __forceinline__ float gelu_erf_f32(float x) {
    const float ax = fabsf(x), z = ax * 0.70710678118654752f;
    const float t = __builtin_amdgcn_rcpf(fmaf(0.3275911f, z, 1.0f));
    const float poly = t * fmaf(t, fmaf(t, fmaf(t, fmaf(t, 1.061405429f, -1.453152027f), 1.421413741f), -0.284496736f), 0.254829592f);
    const float g = __builtin_amdgcn_exp2f(z * z * -1.4426950408889634f);     // exp(-z^2)
    return fmaxf(x, 0.0f) - 0.5f * __builtin_amdgcn_fmed3f(ax, 0.0f, 20.0f) * (poly * g);
}

// splitmix64's output function: the per-word mixer of the streamed-bytes checksum.
__device__ __forceinline__ uint64_t cf_mix64(uint64_t z) {
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}
constexpr uint64_t CF_GOLDEN64 = 0x9E3779B97F4A7C15ull;
