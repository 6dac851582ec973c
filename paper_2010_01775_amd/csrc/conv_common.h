// Element types, conversions and activations that the convolution kernels
// share, and the interface of the 8/16-bit tile kernels (conv_tile.h).
#pragma once

#include <math.h>

#include "npg_internal.h"

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef long fp8x8;  // eight e4m3 bytes

// K chunks of the matrix-core tiles (input channels staged at a time)
constexpr int KC32 = 16;  // input channels per chunk, FP32 path
constexpr int KC16 = 32;  // input channels per chunk, BF16 path
constexpr int KC16S = 16; // BF16 path for 16- and 48-channel inputs: one 32-wide
                          // MFMA K slice covers two taps of 16 channels
constexpr int KC8 = 32;   // FP8 path, as BF16
constexpr int KC8S = 16;
constexpr float E4M3_MAX = 448.0f;

// OCP FP8 e4m3: 1 sign, 4 exponent bits (bias 7), 3 mantissa bits, no
// infinities, 0x7f / 0xff NaN, largest finite 448, subnormal step 2^-9.
// Encoding rounds to nearest even and saturates at +-448.
__host__ __device__ inline uint8_t e4m3_enc(float x) {
  if (x != x) return 0x7f;
  uint8_t s = 0;
  if (x < 0.0f) {
    s = 0x80;
    x = -x;
  }
  if (x >= E4M3_MAX) return s | 0x7e;
  if (x < 0.015625f) return s | (uint8_t)rintf(x * 512.0f);  // subnormal (8 -> 0x08, the smallest normal)
  int e;
  (void)frexpf(x, &e);                          // x in [2^(e-1), 2^e)
  int m = (int)rintf(ldexpf(x, 4 - e)) - 8;     // mantissa steps of 2^(e-4), in [0, 8]
  int E = e - 1 + 7;
  if (m == 8) {
    m = 0;
    ++E;
  }
  return s | (uint8_t)((E << 3) | m);  // x < 448 keeps (E, m) <= (15, 6)
}
__host__ __device__ inline float e4m3_dec(uint8_t v) {
  const int e = (v >> 3) & 15, m = v & 7;
  float mag = e ? ldexpf((float)(8 + m), e - 10) : ldexpf((float)m, -9);
  if ((v & 0x7f) == 0x7f) mag = NAN;
  return (v & 0x80) ? -mag : mag;
}

// Device forms on the conversion instructions (gfx950 converts to OCP e4m3
// with round to nearest even; out-of-range inputs, which would give NaN,
// are clamped first so that both forms saturate alike).
__device__ __forceinline__ uint8_t e4m3_enc_d(float x) {
  const float c = x != x ? x : fminf(fmaxf(x, -E4M3_MAX), E4M3_MAX);
  return (uint8_t)(__builtin_amdgcn_cvt_pk_fp8_f32(c, c, 0, false) & 0xff);
}
__device__ __forceinline__ float e4m3_dec_d(uint8_t v) { return __builtin_amdgcn_cvt_f32_fp8((int)v, 0); }
// Four values as four e4m3 bytes (first value in the low byte), each clamped
// and rounded as e4m3_enc_d does: two conversion instructions.
__device__ __forceinline__ float e4m3_clamp_d(float x) { return x != x ? x : fminf(fmaxf(x, -E4M3_MAX), E4M3_MAX); }
__device__ __forceinline__ uint32_t e4m3_pack4_d(float a, float b, float c, float d) {
  const int lo = __builtin_amdgcn_cvt_pk_fp8_f32(e4m3_clamp_d(a), e4m3_clamp_d(b), 0, false);
  return (uint32_t)__builtin_amdgcn_cvt_pk_fp8_f32(e4m3_clamp_d(c), e4m3_clamp_d(d), lo, true);
}

enum Act : int { ACT_RELU = 0, ACT_SOFTPLUS = 1, ACT_ELU = 2 };

// ReLU, or ELU (Clevert et al. 2016: x for x > 0, e^x - 1 otherwise).
template <class A>
__device__ __forceinline__ A act_fn(A v, int act) {
  if (act == ACT_ELU) {
    if constexpr (sizeof(A) == 8)
      return v > (A)0 ? v : (A)expm1((double)v);
    else
      return v > (A)0 ? v : (A)expm1f((float)v);
  }
  return v > (A)0 ? v : (A)0;
}

__device__ __forceinline__ float bf2f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

// float -> bf16 bits, round to nearest even (one conversion instruction)
__device__ __forceinline__ uint16_t f2bf(float f) { return __builtin_bit_cast(uint16_t, (__bf16)f); }

__device__ __forceinline__ float softplus_f(float x) { return fmaxf(x, 0.0f) + log1pf(expf(-fabsf(x))); }
__device__ __forceinline__ double softplus_f(double x) { return fmax(x, 0.0) + log1p(exp(-fabs(x))); }

// activation storage types: double (FP32 mode) and bf16 bits (BF16 mode)
template <class T> __device__ __forceinline__ double to_d(T v);
template <> __device__ __forceinline__ double to_d<double>(double v) { return v; }
template <> __device__ __forceinline__ double to_d<float>(float v) { return v; }
template <> __device__ __forceinline__ double to_d<uint16_t>(uint16_t v) { return bf2f(v); }
template <> __device__ __forceinline__ double to_d<uint8_t>(uint8_t v) { return e4m3_dec_d(v); }
template <class T> __device__ __forceinline__ T from_d(double v);
template <> __device__ __forceinline__ double from_d<double>(double v) { return v; }
template <> __device__ __forceinline__ float from_d<float>(double v) { return (float)v; }
template <> __device__ __forceinline__ uint16_t from_d<uint16_t>(double v) { return f2bf((float)v); }
template <> __device__ __forceinline__ uint8_t from_d<uint8_t>(double v) { return e4m3_enc_d((float)v); }

// Buffer-resource word 3 for raw (unswizzled, untyped) buffers on gfx9.
constexpr int BUF_WORD3 = 0x00020000;
typedef __attribute__((address_space(3))) void lds_void;
constexpr size_t DMA_BLOCK = 1024;  // bytes one LDS load instruction writes
