// The truncated exponential series in shifted form, and the matrix-core and
// bfloat16 helpers of the kernels that evaluate attention pair by pair.
//
// With m = P - 1, v = s + 1 and a_j = (m! / j!) sum_{r <= m - j} (-1)^r / r!,
//     m! f_P(s) = v^m + a_{m-2} v^{m-2} + ... + a_0
// (a_m = 1, and a_{m-1} = 0 because the shift by 1 removes it): one product and
// sum fewer than the series itself, for instance 6 f_4 = v (v^2 + 3) + 2.  The
// shift is free: the score r = q.k comes out of the matrix cores with
// sqrt(d_k) as the accumulator's start, u = r + sqrt(d_k) = v sqrt(d_k), and
//     kappa f_P = u^m + e_{m-2} u^{m-2} + ... + e_0,  e_j = a_j d_k^((m-j)/2),
//     kappa = m! d_k^(m/2).
// The factor kappa is the same for every pair and leaves with the
// normalisation.  It is up to 1e10 (P = 8, d_k = 64) and would take as much from
// the range of the scores, so r comes in units of 2^x (one operand's rows are
// scaled, exactly), with 2^x near kappa^(1/m): then all of u, e_j and the sum are
// scaled by powers of two, the results are the same bits, and the factor left on
// f_P is within 2^(+-m/2).
#pragma once

#include <hip/hip_runtime.h>

#include <cmath>
#include <type_traits>
#include <utility>

#include "device_common.hpp"

namespace sata {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned short u16;

constexpr int kMaxSeries = 8;  // terms

struct Series {
  float e[kMaxSeries];   // e[j] of f_P
  float de[kMaxSeries];  // e[j] of f_{P-1} (the derivative's)
  float shift;           // sqrt(d_k)
  float scale;           // 2^-x: of the queries (or keys) that make the scores
};

inline Series make_series(int P, int dk) {
  Series se{};
  double kappa = 1.0;
  for (int j = 1; j < P; ++j) kappa *= j * std::sqrt((double)dk);
  const int x = P > 1 ? (int)std::lround(std::log2(kappa) / (P - 1)) : 0;
  auto fill = [&](int m, float* e) {
    double fact[kMaxSeries];  // m! / j!
    fact[m] = 1.0;
    for (int j = m - 1; j >= 0; --j) fact[j] = fact[j + 1] * (j + 1);
    for (int j = 0; j <= m; ++j) {
      double a = 0.0, t = 1.0;
      for (int r = 0; r <= m - j; ++r) {
        a += t;
        t /= -(r + 1);
      }
      if (j == m - 1) a = 0.0;  // (1 - 1)
      e[j] = std::ldexp((float)(fact[j] * a * std::pow((double)dk, 0.5 * (m - j))), -x * (m - j));
    }
  };
  fill(P - 1, se.e);
  if (P > 1) fill(P - 2, se.de);
  se.shift = std::ldexp((float)std::sqrt((double)dk), -x);
  se.scale = std::ldexp(1.f, -x);
  return se;
}

// w[i] = kappa f(u[i]) of degree m >= 1 from the coefficients e; MM = m when
// it is known at compile time, else 0: then one pass over all N values per
// term, its coefficient read from lane j of `lanes` (branches per few values,
// or all degrees' code beside each other, ran at a third of this rate).
template <int MM, int N>
__device__ __forceinline__ void series_eval(int m, const float (&u)[N], float (&w)[N], const float (&e)[kMaxSeries],
                                            float lanes) {
  if constexpr (MM == 1) {
#pragma unroll
    for (int i = 0; i < N; ++i) w[i] = u[i];
  } else if constexpr (MM > 1) {
#pragma unroll
    for (int i = 0; i < N; ++i) {
      float r = fmaf(u[i], u[i], e[MM - 2]);
#pragma unroll
      for (int j = MM - 3; j >= 0; --j) r = fmaf(r, u[i], e[j]);
      w[i] = r;
    }
  } else {
    if (m == 0) {
#pragma unroll
      for (int i = 0; i < N; ++i) w[i] = 1.f;
      return;
    }
    if (m == 1) {
#pragma unroll
      for (int i = 0; i < N; ++i) w[i] = u[i];
      return;
    }
    auto c = [&](int j) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(lanes), j)); };
    float r[N];
    const float c2 = c(m - 2);
#pragma unroll
    for (int i = 0; i < N; ++i) r[i] = fmaf(u[i], u[i], c2);
#pragma unroll 1
    for (int j = m - 3; j >= 0; --j) {
      const float cj = c(j);
#pragma unroll
      for (int i = 0; i < N; ++i) r[i] = fmaf(r[i], u[i], cj);
    }
#pragma unroll
    for (int i = 0; i < N; ++i) w[i] = r[i];
  }
}

__device__ __forceinline__ uint32_t pack2(float lo, float hi) {
  bf16x2 v;
  v[0] = (__bf16)lo;
  v[1] = (__bf16)hi;
  return __builtin_bit_cast(uint32_t, v);
}
__device__ __forceinline__ float lo_f32(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float hi_f32(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

// eight consecutive values as one bf16 operand; x becomes what it leaves out
__device__ __forceinline__ uint4 to_bf16(const float* x) {
  return uint4{pack2(x[0], x[1]), pack2(x[2], x[3]), pack2(x[4], x[5]), pack2(x[6], x[7])};
}
__device__ __forceinline__ void take_bf16(const uint4& w, float* x) {
  const uint32_t u[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    x[2 * i] -= lo_f32(u[i]);
    x[2 * i + 1] -= hi_f32(u[i]);
  }
}

__device__ __forceinline__ f32x4 mfma_bf16(const uint4& a, const uint4& b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0,
                                                 0);
}
__device__ __forceinline__ f32x4 mfma_f32(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// Eight idle cycles between matrix instructions and a branch behind which vector
// instructions read or overwrite their results.  The result of a 16x16x32 takes
// that long; the compiler (ROCm 7.2) keeps the distance inside a block of code,
// but across a branch it was seen to leave 2 and 5 to 7 (three of four rows of
// dk were stale where it was 2).
__device__ __forceinline__ void settle_mfma() {
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("s_nop 7");
  __builtin_amdgcn_sched_barrier(0);
}

// The same for the results r: what reads them comes after, other code may move.
template <int N>
__device__ __forceinline__ void settle_mfma(f32x4 (&r)[N]) {
  static_assert(N <= 4, "operands of the statement");
  if constexpr (N == 1) asm volatile("s_nop 7" : "+v"(r[0]));
  else if constexpr (N == 2) asm volatile("s_nop 7" : "+v"(r[0]), "+v"(r[1]));
  else if constexpr (N == 3) asm volatile("s_nop 7" : "+v"(r[0]), "+v"(r[1]), "+v"(r[2]));
  else asm volatile("s_nop 7" : "+v"(r[0]), "+v"(r[1]), "+v"(r[2]), "+v"(r[3]));
}

// Operand of 8 rows' entries of one column from bf16 rows in LDS, read
// transposed: p and p + next point at this lane's 8 bytes of the first and the
// second four rows (lane l of each 16: row l / 4, columns 4 (l % 4) .. +3; it
// receives column l).
__device__ __forceinline__ uint4 read_transposed(const u16* p, int next) {
  const bf16x4 a = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((__attribute__((address_space(3))) bf16x4*)p);
  const bf16x4 b = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((__attribute__((address_space(3))) bf16x4*)(p + next));
  return __builtin_bit_cast(uint4, (bf16x8)__builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7));
}

// A tensor of `bytes` bytes (below 2^31) read by 16-byte vectors at byte
// offsets; a vector past the end (kNoVector among them) reads as zero, so a
// ragged last chunk needs no test of its own.
constexpr uint32_t kNoVector = 0x80000000u;
struct VectorReader {
  __amdgpu_buffer_rsrc_t rsrc;
  __device__ __forceinline__ VectorReader() = default;
  __device__ __forceinline__ VectorReader(const void* p, int64_t bytes)
      : rsrc(__builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)bytes, 0x00020000)) {}
  // sizeof(V) = 4 or 8 bytes at an offset that is a multiple of them
  template <typename V>
  __device__ __forceinline__ V part(uint32_t offset) const {
    typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
    if constexpr (sizeof(V) == 4)
      return __builtin_bit_cast(V, (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(rsrc, (int)offset, 0, 0));
    else
      return __builtin_bit_cast(V, (u32x2)__builtin_amdgcn_raw_buffer_load_b64(rsrc, (int)offset, 0, 0));
  }
  __device__ __forceinline__ uint4 operator()(uint32_t offset) const {
    typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
    return __builtin_bit_cast(uint4, (u32x4)__builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)offset, 0, 0));
  }
};

// f(integral_constant<int, I>) for I = 0 .. N-1, unrolled.
template <typename F, int... I>
__device__ __forceinline__ void static_for_impl(F&& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  static_for_impl(f, std::make_integer_sequence<int, N>{});
}

}  // namespace sata
