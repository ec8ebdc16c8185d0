// Device-side helpers shared by the HIP kernels (gfx950, wave64).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace rag {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float floatx4;
typedef __attribute__((ext_vector_type(16))) float floatx16;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
typedef __attribute__((address_space(3))) void lds_void_t;

constexpr int kWave = 64;
constexpr int kTile = 64;     // attention tile edge (rows / cols of a score tile)
constexpr int kHeadDim = 64;  // head dimension the attention kernels are built for

// Status-word bits (mirrors the public enum).
constexpr int kDataNegLength = 1, kDataLongLength = 2, kDataTokenCount = 4, kDataQktCap = 8,
              kDataAvCap = 16, kDataScoreCap = 32;

// Variable-sized batched GEMM: output tile, size limits and status-word bits
// (mirror the public constants).
constexpr int kVgemmTileM = 128, kVgemmTileN = 256, kVgemmMaxBatch = 4096, kVgemmMaxDim = 65536;
constexpr int kVgemmNegSize = 1, kVgemmLargeSize = 2, kVgemmTileCap = 4, kVgemmOperandCap = 8,
              kVgemmBf16Shape = 16;

__device__ __forceinline__ float bf16_to_f32(uint16_t b) {
    return __uint_as_float(static_cast<uint32_t>(b) << 16);
}

typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;

// Round to nearest, ties to even (gfx950's v_cvt_pk_bf16_f32, branch-free).
__device__ __forceinline__ uint16_t f32_to_bf16(float f) { return __builtin_bit_cast(uint16_t, static_cast<__bf16>(f)); }

__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
    const bf16x2 v = {static_cast<__bf16>(lo), static_cast<__bf16>(hi)};
    return __builtin_bit_cast(uint32_t, v);
}

// Low / high bf16 halves of a packed pair, widened.
__device__ __forceinline__ float lo_bf16(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float hi_bf16(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

// Workgroup-uniform values made so explicitly: the compiler cannot keep plan reads
// in scalar registers where the same kernel may write the status word (atomicOr),
// and a buffer descriptor built from a per-lane value becomes a per-lane loop.
__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ int64_t uni64(int64_t v) {
    const uint32_t lo = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(v));
    const uint32_t hi = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(static_cast<uint64_t>(v) >> 32));
    return static_cast<int64_t>((static_cast<uint64_t>(hi) << 32) | lo);
}

// All-reduce within aligned groups of G lanes (a power of two), by moves inside the
// vector unit: quad permutes and mirrors inside a row of 16 lanes, then lane swaps
// between rows and between the half waves.  (Shuffles go through the LDS unit, about
// 100 cycles each: a row softmax's 12 in a chain were most of its time.)
template <int CTRL>
__device__ __forceinline__ float dpp_move(float v) {
    return __uint_as_float(__builtin_amdgcn_update_dpp(0u, __float_as_uint(v), CTRL, 0xf, 0xf, true));
}

template <int G, typename Op>
__device__ __forceinline__ float group_reduce(float v, Op op) {
    static_assert(G == 1 || G == 2 || G == 4 || G == 8 || G == 16 || G == 32 || G == 64, "group size");
    if constexpr (G >= 2) v = op(v, dpp_move<0xb1>(v));    // quad_perm 1, 0, 3, 2
    if constexpr (G >= 4) v = op(v, dpp_move<0x4e>(v));    // quad_perm 2, 3, 0, 1
    if constexpr (G >= 8) v = op(v, dpp_move<0x141>(v));   // half-row mirror: the other quad of 8
    if constexpr (G >= 16) v = op(v, dpp_move<0x140>(v));  // row mirror: the other 8 of 16
    if constexpr (G >= 32) {
        const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
        v = op(__uint_as_float(r[0]), __uint_as_float(r[1]));
    }
    if constexpr (G >= 64) {
        const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
        v = op(__uint_as_float(r[0]), __uint_as_float(r[1]));
    }
    return v;
}

template <int G>
__device__ __forceinline__ float group_max(float v) {
    return group_reduce<G>(v, [](float a, float b) { return fmaxf(a, b); });
}
template <int G>
__device__ __forceinline__ float group_sum(float v) {
    return group_reduce<G>(v, [](float a, float b) { return a + b; });
}

__device__ __forceinline__ float wave_max(float v) { return group_max<kWave>(v); }
__device__ __forceinline__ float wave_sum(float v) { return group_sum<kWave>(v); }

__device__ __forceinline__ float gelu_erf(float x) { return 0.5f * x * (1.0f + erff(x * 0.70710678118654752f)); }

__device__ __forceinline__ float gelu_tanh(float x) {
    const float c = 0.79788456080286536f;  // sqrt(2/pi)
    return 0.5f * x * (1.0f + tanhf(c * (x + 0.044715f * x * x * x)));
}

template <int ACT>
__device__ __forceinline__ float activate(float x) {
    if constexpr (ACT == 1) return gelu_erf(x);
    else if constexpr (ACT == 2) return gelu_tanh(x);
    else return x;
}

// GELU (erf form) for bf16 outputs with a branch-free erfc: Abramowitz & Stegun,
// Handbook of Mathematical Functions, formula 7.1.26, erfc(z) ~ t*(a1 + t*(a2 +
// t*(a3 + t*(a4 + t*a5)))) * exp(-z^2), t = 1/(1 + p z), z >= 0, |error| <= 1.5e-7
// (far below bf16 resolution).  Since x*erf(x/sqrt2) is even in x,
// x*Phi(x) = max(x, 0) - |x| * erfc(|x|/sqrt2) / 2, which needs no sign branch and
// keeps the relative accuracy of the small negative branch; the 1/2 is folded into
// the coefficients and exp(-x^2/2) is evaluated as a power of two.
__device__ __forceinline__ float gelu_erf_fast(float x) {
    const float ax = fabsf(x);
    const float t = __builtin_amdgcn_rcpf(fmaf(ax, 0.3275911f * 0.70710678118654752f, 1.0f));
    const float e = __builtin_amdgcn_exp2f(x * x * (-0.5f * 1.4426950408889634f));
    const float half_poly =
        t * (0.5f * 0.254829592f +
             t * (0.5f * -0.284496736f + t * (0.5f * 1.421413741f + t * (0.5f * -1.453152027f + t * (0.5f * 1.061405429f)))));
    return fmaf(-ax, half_poly * e, fmaxf(x, 0.f));
}

template <int ACT>
__device__ __forceinline__ float activate_bf16(float x) {
    if constexpr (ACT == 1) return gelu_erf_fast(x);
    else return activate<ACT>(x);
}

__device__ __forceinline__ floatx4 mfma16x16x32(const bf16x8& a, const bf16x8& b, const floatx4& c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// 32x32x16: lane l supplies row (l % 32) of A and column (l % 32) of B with the 8
// k values 8*(l/32) .. 8*(l/32)+7; it receives C column l % 32, rows
// 8*(r/4) + 4*(l/32) + (r%4) for accumulator element r = 0..15.  Which form is faster
// depends on the operands, since the card is limited by power: chains on registers alone,
// every SIMD at work, reach (TFLOP/s, 32x32x16 and 16x16x32) 2150-2420 and 1980-2200 at
// one wave per SIMD with operands of zeros or ones, but 1680-1730 and 1770-1880 with
// random ones; at two waves per SIMD 1640 and 2230-2330, random 1290-1400 and 1830.  The
// 128 x 256 tiles and smaller ones use this form, the 256 x 256 tiles the other.
__device__ __forceinline__ floatx16 mfma32x32x16(const bf16x8& a, const bf16x8& b, const floatx16& c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ bf16x8 as_bf16x8(const u32x4& v) {
    return __builtin_bit_cast(bf16x8, v);
}

}  // namespace rag
