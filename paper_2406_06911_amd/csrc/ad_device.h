// Device-side helpers shared by the kernel files: vector types, conversions, activations, wavefront reductions, buffer loads.
#pragma once

#include <hip/hip_runtime.h>

namespace ad {

typedef __bf16 bf16;
typedef bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

template <typename T> struct Vec;
template <> struct Vec<bf16> { typedef bf16x8 type; static constexpr int N = 8; };
template <> struct Vec<float> { typedef f32x4 type; static constexpr int N = 4; };

__device__ __forceinline__ float to_f(bf16 v) { return (float)v; }
__device__ __forceinline__ float to_f(float v) { return v; }
template <typename T> __device__ __forceinline__ T from_f(float v);
template <> __device__ __forceinline__ bf16 from_f<bf16>(float v) { return (bf16)v; }
template <> __device__ __forceinline__ float from_f<float>(float v) { return v; }

// x * sigmoid(x) with the hardware reciprocal (1 ulp): the IEEE division the compiler emits for x / (1 + e) by
// default costs about ten vector instructions per element
__device__ __forceinline__ float silu_f(float x) {
  return x * __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(-1.44269504088896341f * x));
}
// Exact-erf GELU x Phi(x):
// gelu(x) = max(x, 0) - |x| erfc(|x| / sqrt 2) / 2 with erfc(z) = (a1 t + ... + a5 t^5) exp(-z^2), t = 1 / (1 + p z) (Abramowitz and
// Stegun 7.1.26, |error| <= 1.5e-7): no sign to put back and no cancellation for negative x.  The GEGLU epilogue is vector work that
// the matrix cores wait for: 17 instructions, two of them transcendental (30 with an IEEE division for t and 1 + erf).  v_rcp_f32 with one
// Newton step instead of the division; |x| is capped where the second term has long underflowed, which keeps infinities out of the
// products.  Against 64 bits over [-12, 12]: largest error 3.3e-7, rms 6.6e-8 (4.7e-7 and 7.2e-8 before).
__device__ __forceinline__ float gelu_f(float x) {
  const float a = fminf(fabsf(x), 100.f);
  const float d = fmaf(0.3275911f * 0.70710678118654752f, a, 1.f);
  const float r = __builtin_amdgcn_rcpf(d);
  const float t = fmaf(fmaf(-d, r, 1.f), r, r);
  const float e = __builtin_amdgcn_exp2f(-0.72134752044448170f * a * a);
  float p = fmaf(t, 0.5f * 1.061405429f, 0.5f * -1.453152027f);
  p = fmaf(t, p, 0.5f * 1.421413741f);
  p = fmaf(t, p, 0.5f * -0.284496736f);
  p = fmaf(t, p, 0.5f * 0.254829592f);
  const float h = 0.5f * x;
  return fmaf(-a, p * t * e, h + fabsf(h));
}

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
// The same on the vector unit alone (all lanes active): rows of 16 lanes by DPP, the four rows through scalar registers.  A shuffle is a round
// trip to the LDS unit, six of them one after the other are a third of a microsecond.
template <int CTRL>
__device__ __forceinline__ float dpp_f(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xf, 0xf, true));
}
__device__ __forceinline__ float lane_f(float v, int lane) {
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), lane));
}
__device__ __forceinline__ float wave_sum_rows(float v) {
  v += dpp_f<0xB1>(v);      // quad_perm 1 0 3 2
  v += dpp_f<0x4E>(v);      // quad_perm 2 3 0 1
  v += dpp_f<0x141>(v);     // row_half_mirror
  v += dpp_f<0x140>(v);     // row_mirror
  return (lane_f(v, 0) + lane_f(v, 16)) + (lane_f(v, 32) + lane_f(v, 48));
}

// Blocks are handed to the 8 XCDs round-robin; renumber them so that consecutive tile ids run on
// the same XCD and share its L2.
__device__ __forceinline__ int xcd_remap(int lid, int nblocks) {
  const int per = nblocks >> 3, rem = nblocks & 7;
  const int xcd = lid & 7, idx = lid >> 3;
  return xcd * per + (xcd < rem ? xcd : rem) + idx;
}

// Division of a 32-bit unsigned by a divisor that is the same for the whole launch (Granlund-Montgomery): the host
// derives a multiplier and two shifts, the device needs a high multiply, a subtract, an add and two shifts.
// Exact for every numerator below 2^32.
struct FastDiv { unsigned mul, sh1, sh2; };
static inline FastDiv make_fastdiv(unsigned d) {
  unsigned l = 0;
  while ((1ull << l) < d) ++l;                                  // ceil(log2 d)
  const unsigned long long m = ((1ull << 32) * ((1ull << l) - d)) / d + 1;
  return FastDiv{(unsigned)m, l < 1 ? l : 1u, l > 0 ? l - 1 : 0u};
}
__device__ __forceinline__ unsigned fast_div(unsigned n, FastDiv f) {
  const unsigned t = __umulhi(f.mul, n);
  return (t + ((n - t) >> f.sh1)) >> f.sh2;
}

// 16-byte loads through a buffer resource: lanes whose offset is kOob (beyond num_records) read zeros
// without touching memory, which is how padding taps and rows past M are produced without branches.
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
constexpr unsigned kOob = 0x80000000u;
__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* base, unsigned bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, (int)bytes, 0x00020000);
}
template <typename V>
__device__ __forceinline__ V buffer_load16(__amdgpu_buffer_rsrc_t r, unsigned voffset, unsigned soffset) {
  const u32x4 raw = __builtin_amdgcn_raw_buffer_load_b128(r, (int)voffset, (int)soffset, 0);
  return __builtin_bit_cast(V, raw);
}

template <typename T> struct Vec4;
template <> struct Vec4<bf16> { typedef bf16x4 type; };
template <> struct Vec4<float> { typedef f32x4 type; };

// 16x16 MFMA on 16-byte fragments: lane (r16, kg) holds row r16 of an operand at the kg-th 16-byte piece of a 64-byte run of K, and of the
// result row r16 of b, columns (rows of a) 4 kg .. 4 kg + 3
template <typename T> struct Mma16;
template <> struct Mma16<bf16> {
  static __device__ __forceinline__ void run(const bf16x8& a, const bf16x8& b, f32x4& c) { c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0); }
};
template <> struct Mma16<float> {
  static __device__ __forceinline__ void run(const f32x4& a, const f32x4& b, f32x4& c) {
#pragma unroll
    for (int e = 0; e < 4; ++e) c = __builtin_amdgcn_mfma_f32_16x16x4f32(a[e], b[e], c, 0, 0, 0);
  }
};

}  // namespace ad
