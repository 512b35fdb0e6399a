// Gradients of the causal prefill pair by pair: with w = f_P(s), w' = f_{P-1}(s)
// of s = q_T . k_t / sqrt(d_k), a = dy_T . v_t, Z_T = sum_t w and
// mu_T = dy_T . y_T = sum_t w a / Z_T,
//     dL/dq_T = sum_t g_Tt k_t,   dL/dk_t = sum_T g_Tt q_T,
//     dL/dv_t = sum_T (w_Tt / Z_T) dy_T,   g = w' (a - mu_T) / (Z_T sqrt(d_k)),
// the gradient of the causal output (App. A2) with the state's contraction over
// features carried out inside f_P.  Work per head-token: about
// (n / 2)(10 d_k + 8 d_v) matrix flops against the state form's
// 10 D (d_v + 1), so it serves all but very long sequences.
//
// Two launches.  backward_rows sweeps the keys of its queries twice: once for
// Z and mu, once for dq.  backward_cols sweeps the queries of its keys for dk
// and dv, with the rows' Z and mu from the first.
//
// Bound: vector instructions (the series and its derivative, and splitting w / Z
// and g into three bfloat16 numbers).  B = 8, H = 32, n = 2048, d = 32, P = 4
// bfloat16: rows 0.42 ms, vector instructions issuing on 72% of a SIMD's cycles,
// matrix cores busy on 27%, 2.9 waves in flight; columns 0.56 ms, 66%, 22% and
// 2.2 waves (the last own rows have few others left to sweep).  The scans take
// 106 ms.
//
// Layout (as prefill_direct.hip): scores transposed so that a lane holds one
// own row (query, or key in backward_cols) and 4 + 4 others of a 32-row step,
// which is the operand layout of the second contraction; the other side's rows
// are staged in LDS as they lie in memory (64 at a time, double buffered) and
// read both along rows (scores) and transposed (contractions).
//
// Precision: float32 throughout, on the bfloat16 matrix cores.  With float32
// inputs a chunk's contractions are summed from zero and then added to the
// running sums (one rounding of those per chunk; without it dk and dv of 777
// tokens were 2 times further off than with float32 sums in chunks).  bfloat16
// inputs are exact operands; float32 values (float32 inputs, w / Z and g) are
// carried as three bfloat16 numbers (24 bits) and a product of two as the six
// partial products of order 2^-16 and up, accumulated in float32.
//
// Values that are not finite stay with the tokens that depend on them.  Only a
// row's own chunk holds masked pairs, and a masked weight's zero times an
// infinity or NaN would reach the sum, so steps of an own chunk look at their
// rows' exponents and, if one is not finite, contract with its entries left out
// (0 to 3% of the time, 9% at most: d_k = 64, P = 4, 128 tokens).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "kernels.hpp"
#include "route.hpp"
#include "series.hpp"

namespace sata {

namespace {

constexpr int kCh = 64;  // rows per staged chunk
constexpr int kNW = 4;   // waves per workgroup

// sum of the products a[i] b[j] with i + j <= 2, smallest first
template <int NA, int NB>
__device__ __forceinline__ f32x4 dot_planes(const uint4 (&a)[NA], const uint4 (&b)[NB], f32x4 c) {
#pragma unroll
  for (int t = 2; t >= 0; --t)
#pragma unroll
    for (int i = 0; i <= t; ++i)
      if (i < NA && t - i < NB) c = mfma_bf16(a[i], b[t - i], c);
  return c;
}

// DT: tiles of 16 covering d_k and d_v.
template <typename T, int DT>
struct BwdLayout {
  static constexpr int kPl = sizeof(T) == 4 ? 3 : 1;  // planes of an input row
  static constexpr int kKS = (DT + 1) / 2;            // contraction steps of 32 over a row
  // bf16 per LDS row: an odd multiple of 8 banks, so that the rows a half wave
  // reads transposed lie in distinct banks
  static constexpr int kRS = kKS == 1 ? 48 : 80;
  static constexpr int kPlane = kCh * kRS;
  static constexpr int kTensor = kPl * kPlane;
  static constexpr int kStat = 3 * kCh * 2;  // u16 of the rows' statistics (backward_cols)
  static constexpr int kBuf = 2 * kTensor + kStat;
  static constexpr int kBytes = 2 * kBuf * 2;
  static constexpr int kEV = 16 / sizeof(T);
  static constexpr int kIt = (kCh * 16 * DT / kEV + kNW * 64 - 1) / (kNW * 64);
};

// One input tensor's rows on their way to LDS: 16-byte vectors where rows
// allow them (width a multiple of a vector, base aligned), else elements.
template <typename T, int DT>
struct RowStage {
  using L = BwdLayout<T, DT>;
  const T* base;
  int n, width;
  bool vec;
  VectorReader read;
  uint4 r[L::kIt];
  int at[L::kIt];       // where a vector goes in a plane (-1: past the rows)
  uint32_t from[L::kIt];  // where it comes from in a chunk

  __device__ void init(const T* p, int n_, int width_) {
    base = p;
    n = n_;
    width = width_;
    read = VectorReader(p, (int64_t)n * width * sizeof(T));
    const int nv = width / L::kEV;
    vec = width % L::kEV == 0 && ((uintptr_t)p & 15) == 0;
#pragma unroll
    for (int i = 0; i < L::kIt; ++i) {
      const int idx = threadIdx.x + i * kNW * 64;
      const bool on = vec && idx < kCh * nv;
      at[i] = on ? (idx / nv) * L::kRS + idx % nv * L::kEV : -1;
      from[i] = on ? 16u * idx : kNoVector;
    }
  }
  // zero what staging never writes: columns past the width
  __device__ void clear(u16* dst) const {
    const int pad = 32 * L::kKS - width;
    for (int pl = 0; pl < L::kPl; ++pl)
      for (int i = threadIdx.x; i < kCh * pad; i += kNW * 64)
        dst[pl * L::kPlane + (i / pad) * L::kRS + width + i % pad] = 0;
  }
  __device__ void fetch(int c) {
    const uint32_t chunk = (uint32_t)c * (uint32_t)(kCh * width * (int)sizeof(T));
#pragma unroll
    for (int i = 0; i < L::kIt; ++i) r[i] = read(from[i] + chunk);
  }
  __device__ float entry(int row, int col) const {
    const T x = base[(int64_t)row * width + col];
    if constexpr (sizeof(T) == 4) return x;
    else return __uint_as_float((uint32_t)x << 16);
  }
  __device__ static void put_elem(u16* dst, T x) {
    if constexpr (sizeof(T) == 4) {
      float f = x;
#pragma unroll
      for (int pl = 0; pl < L::kPl; ++pl) {
        const uint32_t h = pack2(f, 0.f);
        dst[pl * L::kPlane] = (u16)h;
        f -= lo_f32(h);
      }
    } else {
      dst[0] = x;
    }
  }
  __device__ void put(u16* dst, int c) const {
    if (vec) {
#pragma unroll
      for (int i = 0; i < L::kIt; ++i) {
        if (at[i] < 0) continue;
        if constexpr (sizeof(T) == 4) {
          float x[4] = {__uint_as_float(r[i].x), __uint_as_float(r[i].y), __uint_as_float(r[i].z),
                        __uint_as_float(r[i].w)};
#pragma unroll
          for (int pl = 0; pl < L::kPl; ++pl) {
            const uint2 h = {pack2(x[0], x[1]), pack2(x[2], x[3])};
            *(uint2*)(dst + pl * L::kPlane + at[i]) = h;
            x[0] -= lo_f32(h.x), x[1] -= hi_f32(h.x), x[2] -= lo_f32(h.y), x[3] -= hi_f32(h.y);
          }
        } else {
          *(uint4*)(dst + at[i]) = r[i];
        }
      }
    } else {
      const int rows = min(kCh, n - c * kCh);
      const T* const s = base + (int64_t)c * kCh * width;
      for (int i = threadIdx.x; i < kCh * width; i += kNW * 64) {
        const int row = i / width;
        put_elem(dst + row * L::kRS + i - row * width, row < rows ? s[i] : (T)0);
      }
    }
  }
};

// B operands of one own row per lane times a power of two: entries 32 ks + 8 g4
// .. +7, all planes.
template <typename T, int DT>
__device__ __forceinline__ void load_own(const T* p, bool ok, int width, int g4, float scale,
                                         uint4 (&f)[BwdLayout<T, DT>::kKS][BwdLayout<T, DT>::kPl]) {
  using L = BwdLayout<T, DT>;
#pragma unroll
  for (int ks = 0; ks < L::kKS; ++ks) {
    const int c0 = 32 * ks + 8 * g4;
    if constexpr (sizeof(T) == 4) {
      float x[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) x[j] = ok && c0 + j < width ? p[c0 + j] * scale : 0.f;
#pragma unroll
      for (int pl = 0; pl < L::kPl; ++pl) {
        f[ks][pl] = to_bf16(x);
        take_bf16(f[ks][pl], x);
      }
    } else {
      uint32_t u[4] = {0u, 0u, 0u, 0u};
#pragma unroll
      for (int j = 0; j < 8; ++j)
        if (ok && c0 + j < width) u[j >> 1] |= (uint32_t)p[c0 + j] << (16 * (j & 1));
#pragma unroll
      for (int j = 0; j < 4; ++j) u[j] = pack2(lo_f32(u[j]) * scale, hi_f32(u[j]) * scale);
      f[ks][0] = uint4{u[0], u[1], u[2], u[3]};
    }
  }
}

// A operands of 16 staged rows: entries 32 ks + 8 g4 .. +7 of row l15, all planes.
template <typename T, int DT>
__device__ __forceinline__ void load_rows(const u16* rows, int l15, int g4,
                                          uint4 (&f)[BwdLayout<T, DT>::kKS][BwdLayout<T, DT>::kPl]) {
  using L = BwdLayout<T, DT>;
#pragma unroll
  for (int ks = 0; ks < L::kKS; ++ks)
#pragma unroll
    for (int pl = 0; pl < L::kPl; ++pl)
      f[ks][pl] = *(const uint4*)(rows + pl * L::kPlane + l15 * L::kRS + 32 * ks + 8 * g4);
}

template <int KS, int PL>
__device__ __forceinline__ f32x4 dot_rows(const uint4 (&a)[KS][PL], const uint4 (&b)[KS][PL], float start) {
  f32x4 c = {start, start, start, start};
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) c = dot_planes(a[ks], b[ks], c);
  return c;
}
// Scores: with three planes the shift is added to the products' sum (with it first,
// rounded with at every product, dv of n = 9743, d = 48, P = 3 was 6% further from
// 64 bits than with the scans, of n = 658, d = 64, P = 2 5%), but for P = 4 of the
// widest rows, which have no registers for it and are 2 to 4 times nearer than the
// scans without.
template <int PL, int DT, int PP>
constexpr bool shift_last() {
  return PL > 1 && !(DT == 4 && PP == 4);
}

// Eight float32 values as three bf16 operands.
__device__ __forceinline__ void split3(float (&x)[8], uint4 (&b)[3]) {
#pragma unroll
  for (int pl = 0; pl < 3; ++pl) {
    b[pl] = to_bf16(x);
    if (pl < 2) take_bf16(b[pl], x);
  }
}

// The entries of a plane that are infinite or NaN, all bits of each set.
__device__ __forceinline__ uint4 not_finite_entries(const uint4& w) {
  auto wide = [](uint32_t x) { return ((((x & 0x7f807f80u) + 0x00800080u) & 0x80008000u) >> 15) * 0xffffu; };
  return uint4{wide(w.x), wide(w.y), wide(w.z), wide(w.w)};
}

// acc[j] += (column tile j of the staged rows 32 s .. +31)^T times b; entries
// that are not finite count as zero if `clean`
template <typename T, int DT>
__device__ __forceinline__ void contract(const u16* rows, int s, int l15, int g4, const uint4 (&b)[3],
                                         f32x4 (&acc)[DT], bool clean = false) {
  using L = BwdLayout<T, DT>;
  const u16* const p = rows + (32 * s + 4 * g4 + (l15 >> 2)) * L::kRS + 4 * (l15 & 3);
#pragma unroll
  for (int j = 0; j < DT; ++j) {
    uint4 a[L::kPl];
#pragma unroll
    for (int pl = 0; pl < L::kPl; ++pl) a[pl] = read_transposed(p + pl * L::kPlane + 16 * j, 16 * L::kRS);
    if (__builtin_expect(clean, 0)) {
      const uint4 m = not_finite_entries(a[0]);
#pragma unroll
      for (int pl = 0; pl < L::kPl; ++pl) a[pl].x &= ~m.x, a[pl].y &= ~m.y, a[pl].z &= ~m.z, a[pl].w &= ~m.w;
    }
    acc[j] = dot_planes(a, b, acc[j]);
  }
}

// Bits set where one of the rows' entries (16 rows in their first plane, as
// load_rows gives them) has the exponent of infinities and NaN.
template <int KS, int PL>
__device__ __forceinline__ uint32_t not_finite(const uint4 (&f)[KS][PL]) {
  uint32_t bits = 0;
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) {
    const uint32_t w[4] = {f[ks][0].x, f[ks][0].y, f[ks][0].z, f[ks][0].w};
#pragma unroll
    for (int i = 0; i < 4; ++i) bits |= (w[i] & 0x7f807f80u) + 0x00800080u;
  }
  return bits & 0x80008000u;
}

// Where a chunk's contractions are summed: in `chunk`, from zero, with three
// planes; else in the running sums themselves.
template <int PL, int DT>
__device__ __forceinline__ f32x4 (&chunk_sum(f32x4 (&chunk)[DT], f32x4 (&acc)[DT]))[DT] {
  if constexpr (PL == 1) return acc;
  else {
#pragma unroll
    for (int j = 0; j < DT; ++j) chunk[j] = f32x4{0.f, 0.f, 0.f, 0.f};
    return chunk;
  }
}
template <int PL, int DT>
__device__ __forceinline__ void add_chunk(f32x4 (&chunk)[DT], f32x4 (&acc)[DT]) {
  if constexpr (PL > 1) {
    settle_mfma(chunk);
#pragma unroll
    for (int j = 0; j < DT; ++j) acc[j] += chunk[j];
  }
}

// Long sums of float32 dk and dv move on to the output every kFlush chunks, so
// that their terms are not all rounded at full length (dk of n = 16000, d = 32,
// P = 4 was 3% further from 64 bits than with the scans; wider rows, which have
// no registers for it, take few features to the scans before that).
constexpr int kFlush = 32;
template <typename T, int DT>
constexpr bool flushes() {
  return sizeof(T) == 4 && DT <= 2;
}
template <int DT>
__device__ __forceinline__ void flush_row(float* p, int width, int g4, f32x4 (&acc)[DT], bool first) {
#pragma unroll
  for (int j = 0; j < DT; ++j)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int c = 16 * j + 4 * g4 + r;
      if (c < width) p[c] = first ? acc[j][r] : p[c] + acc[j][r];
      acc[j][r] = 0.f;
    }
}

// lane (l15, g4): columns 16 j + 4 g4 .. +3 of one own row; `more`: plus what the
// row holds already
template <typename T, int DT>
__device__ __forceinline__ void store_row(T* p, int width, int g4, const f32x4 (&acc)[DT], float scale,
                                          bool more = false) {
  settle_mfma();
#pragma unroll
  for (int j = 0; j < DT; ++j)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int c = 16 * j + 4 * g4 + r;
      if (c < width) {
        if constexpr (flushes<T, DT>()) p[c] = (more ? p[c] + acc[j][r] : acc[j][r]) * scale;
        else if constexpr (sizeof(T) == 4) p[c] = acc[j][r] * scale;
        else p[c] = f32_to_bf16(acc[j][r] * scale).bits;
      }
    }
}

struct BwdArgs {
  const void *q, *k, *v, *dy;
  void *dq, *dk, *dv;
  float* stat;  // [head][chunk][3][64]: 1 / Z, (P-1) / Z, -mu (P-1) / Z (in the series' units)
  Series se;
  int heads, n, dk_, dv_, P, blocks, by_xcd;
};

// blockIdx -> (head, block): each XCD takes whole heads where there are 8 or
// more, so that a head's rows are read through one L2.
__device__ __forceinline__ bool locate(const BwdArgs& a, int& head, int& blk) {
  if (a.by_xcd) {
    const int j = blockIdx.x >> 3;
    head = (j / a.blocks) * 8 + (int)(blockIdx.x & 7);
    blk = j % a.blocks;
    return head < a.heads;
  }
  head = blockIdx.x % a.heads;
  blk = blockIdx.x / a.heads;
  return true;
}

// (waves per SIMD: as many as the working registers allow without the rare
// handling of values that are not finite)
template <typename T, int DT, int NQ, int PP>
__global__ void __launch_bounds__(kNW * 64, sizeof(T) == 2 ? 3 : 2) backward_rows(BwdArgs a) {
  using L = BwdLayout<T, DT>;
  extern __shared__ __attribute__((aligned(16))) u16 smem16[];
  const int tid = threadIdx.x, lane = tid & 63, l15 = lane & 15, g4 = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int head, blk;
  if (!locate(a, head, blk)) return;
  blk = a.blocks - 1 - blk;  // the longest sweeps first
  const int n = a.n, dk = a.dk_, dv = a.dv_, m = a.P - 1;
  const float lw = lane < kMaxSeries ? a.se.e[lane & 7] : 0.f, ld = lane < kMaxSeries ? a.se.de[lane & 7] : 0.f;
  constexpr int MM = PP > 0 ? PP - 1 : 0, DM = PP > 1 ? PP - 2 : 0;
  constexpr bool kLast = shift_last<L::kPl, DT, PP>();
  const T* const qp = (const T*)a.q + (int64_t)head * n * dk;
  const T* const dyp = (const T*)a.dy + (int64_t)head * n * dv;
  RowStage<T, DT> sk, sv;
  sk.init((const T*)a.k + (int64_t)head * n * dk, n, dk);
  sv.init((const T*)a.v + (int64_t)head * n * dv, n, dv);
  const int nch = (n + kCh - 1) / kCh;
  const int c_first = blk * NQ, chunks = min(c_first + NQ, nch);
  for (int b = 0; b < 2; ++b) {
    sk.clear(smem16 + b * L::kBuf);
    sv.clear(smem16 + b * L::kBuf + L::kTensor);
  }
  uint4 qf[NQ][L::kKS][L::kPl], df[NQ][L::kKS][L::kPl];
#pragma unroll
  for (int i = 0; i < NQ; ++i) {
    const int row = (c_first + i) * kCh + 16 * wave + l15;
    load_own<T, DT>(qp + (int64_t)row * dk, row < n, dk, g4, a.se.scale, qf[i]);
    load_own<T, DT>(dyp + (int64_t)row * dv, row < n, dv, g4, 1.f, df[i]);
  }
  // work(K rows, V rows, tile, on its own chunk) for every key chunk and query tile
  auto sweep = [&](auto&& work) {
    sk.fetch(0);
    sv.fetch(0);
    sk.put(smem16, 0);
    sv.put(smem16 + L::kTensor, 0);
    __syncthreads();
    for (int c = 0; c < chunks; ++c) {
      if (c + 1 < chunks) {
        sk.fetch(c + 1);
        sv.fetch(c + 1);
      }
      const u16* const kb = smem16 + (c & 1) * L::kBuf;
      const u16* const vb = kb + L::kTensor;
      static_for<NQ>([&](auto ic) {
        constexpr int I = decltype(ic)::value;
        if (c < c_first + I) work(kb, vb, ic, std::false_type{});
        else if (c == c_first + I) work(kb, vb, ic, std::true_type{});
      });
      if (c + 1 < chunks) {
        sk.put(smem16 + ((c + 1) & 1) * L::kBuf, c + 1);
        sv.put(smem16 + ((c + 1) & 1) * L::kBuf + L::kTensor, c + 1);
      }
      __syncthreads();
    }
  };
  // u and a of query tile i against keys 32 s .. +31 (4 h + r: key 32 s + 16 h + 4 g4 + r);
  // bad: bits for keys that are not finite
  auto pairs = [&](const u16* kb, const u16* vb, int s, auto ic, float (&u)[8], float (&av)[8], uint32_t& bad) {
    constexpr int I = decltype(ic)::value;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      uint4 f[L::kKS][L::kPl];
      load_rows<T, DT>(kb + (32 * s + 16 * h) * L::kRS, l15, g4, f);
      const f32x4 x = dot_rows(f, qf[I], kLast ? 0.f : a.se.shift);
      bad |= not_finite(f);
      load_rows<T, DT>(vb + (32 * s + 16 * h) * L::kRS, l15, g4, f);
      const f32x4 y = dot_rows(f, df[I], 0.f);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        u[4 * h + r] = kLast ? x[r] + a.se.shift : x[r];
        av[4 * h + r] = y[r];
      }
    }
    if constexpr (MM == 0) settle_mfma();  // (the series branches on its degree)
  };
  auto masked = [&](int s, float (&x)[8]) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (32 * s + 16 * h + 4 * g4 + r > 16 * wave + l15) x[4 * h + r] = 0.f;
  };

  // ---- Z and sum w a
  float z[NQ], ma[NQ];
#pragma unroll
  for (int i = 0; i < NQ; ++i) z[i] = ma[i] = 0.f;
  sweep([&](const u16* kb, const u16* vb, auto ic, auto own) {
    constexpr int I = decltype(ic)::value;
    constexpr bool kOwn = decltype(own)::value;
    const int steps = kOwn ? (wave >> 1) + 1 : 2;
    for (int s = 0; s < steps; ++s) {
      float u[8], av[8], w[8];
      uint32_t bad = 0;
      pairs(kb, vb, s, ic, u, av, bad);
      series_eval<MM>(m, u, w, a.se.e, lw);
      if (kOwn) {
        masked(s, w);
        masked(s, av);  // (0 * av would carry a value that is not finite to earlier queries)
      }
      float zs = 0.f, ms = 0.f;  // (a step's sums first: fewer roundings of the long sums)
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        zs += w[e];
        ms = fmaf(w[e], av[e], ms);
      }
      z[I] += zs;
      ma[I] += ms;
    }
  });
  float mu[NQ], rg[NQ];
  float* const stat = a.stat + (int64_t)head * nch * 3 * kCh;
#pragma unroll
  for (int i = 0; i < NQ; ++i) {
    z[i] += __shfl_xor(z[i], 16);
    z[i] += __shfl_xor(z[i], 32);
    ma[i] += __shfl_xor(ma[i], 16);
    ma[i] += __shfl_xor(ma[i], 32);
    const int c = c_first + i;
    const bool ok = c * kCh + 16 * wave + l15 < n;
    // (z - z: a sum that is not finite leaves no gradient finite, not even 1 / z = 0)
    const float rz = ok ? 1.f / z[i] + (z[i] - z[i]) : 0.f;
    mu[i] = ok ? ma[i] / z[i] : 0.f;
    rg[i] = rz * ((float)m * a.se.scale);
    if (g4 == 0 && c < nch) {
      float* const p = stat + (int64_t)c * 3 * kCh + 16 * wave + l15;
      p[0] = rz;
      p[kCh] = rg[i];
      p[2 * kCh] = -mu[i] * rg[i];
    }
  }

  // ---- dq = (P - 1) / Z sum w' (a - mu) k
  f32x4 acc[NQ][DT];
#pragma unroll
  for (int i = 0; i < NQ; ++i)
#pragma unroll
    for (int j = 0; j < DT; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  sweep([&](const u16* kb, const u16* vb, auto ic, auto own) {
    constexpr int I = decltype(ic)::value;
    constexpr bool kOwn = decltype(own)::value;
    const int steps = kOwn ? (wave >> 1) + 1 : 2;
    f32x4 chunk[DT];
    f32x4(&sum)[DT] = chunk_sum<L::kPl>(chunk, acc[I]);
    for (int s = 0; s < steps; ++s) {
      float u[8], av[8], g[8];
      uint32_t bad = 0;
      pairs(kb, vb, s, ic, u, av, bad);
      series_eval<DM>(m - 1, u, g, a.se.de, ld);
#pragma unroll
      for (int e = 0; e < 8; ++e) g[e] *= av[e] - mu[I];
      if (kOwn) masked(s, g);
      uint4 b[3];
      split3(g, b);
      // (a later key that is not finite times a masked zero is no zero; without
      // it, an earlier one still reaches dq, through g)
      contract<T, DT>(kb, s, l15, g4, b, sum, kOwn && __ballot(bad));
    }
    add_chunk<L::kPl>(chunk, acc[I]);
  });
#pragma unroll
  for (int i = 0; i < NQ; ++i) {
    const int row = (c_first + i) * kCh + 16 * wave + l15;
    if (row < n) store_row<T, DT>((T*)a.dq + ((int64_t)head * n + row) * dk, dk, g4, acc[i], rg[i]);
  }
}

template <typename T, int DT, int NQ, int PP>
__global__ void __launch_bounds__(kNW * 64, sizeof(T) == 2 && DT <= 2 ? (DT == 1 && NQ == 1 ? 4 : 3) : 2)
backward_cols(BwdArgs a) {
  using L = BwdLayout<T, DT>;
  extern __shared__ __attribute__((aligned(16))) u16 smem16[];
  const int tid = threadIdx.x, lane = tid & 63, l15 = lane & 15, g4 = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int head, blk;
  if (!locate(a, head, blk)) return;  // (the first keys have the longest sweeps)
  const int n = a.n, dk = a.dk_, dv = a.dv_, m = a.P - 1;
  const float lw = lane < kMaxSeries ? a.se.e[lane & 7] : 0.f, ld = lane < kMaxSeries ? a.se.de[lane & 7] : 0.f;
  constexpr int MM = PP > 0 ? PP - 1 : 0, DM = PP > 1 ? PP - 2 : 0;
  constexpr bool kLast = shift_last<L::kPl, DT, PP>();
  const T* const kp = (const T*)a.k + (int64_t)head * n * dk;
  const T* const vp = (const T*)a.v + (int64_t)head * n * dv;
  RowStage<T, DT> sq, sy;
  sq.init((const T*)a.q + (int64_t)head * n * dk, n, dk);
  sy.init((const T*)a.dy + (int64_t)head * n * dv, n, dv);
  const int nch = (n + kCh - 1) / kCh;
  const int c_first = blk * NQ;
  const float* const stat = a.stat + (int64_t)head * nch * 3 * kCh;
  for (int b = 0; b < 2; ++b) {
    sq.clear(smem16 + b * L::kBuf);
    sy.clear(smem16 + b * L::kBuf + L::kTensor);
  }
  uint4 kf[NQ][L::kKS][L::kPl], vf[NQ][L::kKS][L::kPl];
  f32x4 dka[NQ][DT], dva[NQ][DT];
#pragma unroll
  for (int i = 0; i < NQ; ++i) {
    const int row = (c_first + i) * kCh + 16 * wave + l15;
    load_own<T, DT>(kp + (int64_t)row * dk, row < n, dk, g4, a.se.scale, kf[i]);
    load_own<T, DT>(vp + (int64_t)row * dv, row < n, dv, g4, 1.f, vf[i]);
#pragma unroll
    for (int j = 0; j < DT; ++j) dka[i][j] = dva[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  float4 rs;
  auto fetch = [&](int c) {
    sq.fetch(c);
    sy.fetch(c);
    if (tid < 3 * kCh / 4) rs = ((const float4*)(stat + (int64_t)c * 3 * kCh))[tid];
  };
  auto put = [&](int b, int c) {
    u16* const base = smem16 + b * L::kBuf;
    sq.put(base, c);
    sy.put(base + L::kTensor, c);
    if (tid < 3 * kCh / 4) ((float4*)(base + 2 * L::kTensor))[tid] = rs;
  };
  bool dirty = false;  // whether own chunks had entries left out
  // key tile i against the queries of a staged chunk
  auto work = [&](const u16* base, [[maybe_unused]] int c, auto ic, auto own) {
    constexpr int I = decltype(ic)::value;
    constexpr bool kOwn = decltype(own)::value;
    const u16* const qb = base;
    const u16* const yb = base + L::kTensor;
    const float* const st = (const float*)(base + 2 * L::kTensor);
    f32x4 ck[DT], cv[DT];
    f32x4(&sumk)[DT] = chunk_sum<L::kPl>(ck, dka[I]);
    f32x4(&sumv)[DT] = chunk_sum<L::kPl>(cv, dva[I]);
    for (int s = kOwn ? wave >> 1 : 0; s < 2; ++s) {
      float u[8], av[8], w[8], g[8];
      uint32_t bad = 0;  // a query or a gradient of the step that is not finite
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        uint4 f[L::kKS][L::kPl];
        load_rows<T, DT>(qb + (32 * s + 16 * h) * L::kRS, l15, g4, f);
        const f32x4 x = dot_rows(f, kf[I], kLast ? 0.f : a.se.shift);
        if (kOwn) bad |= not_finite(f);
        load_rows<T, DT>(yb + (32 * s + 16 * h) * L::kRS, l15, g4, f);
        if (kOwn) bad |= not_finite(f);
        const f32x4 y = dot_rows(f, vf[I], 0.f);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          u[4 * h + r] = kLast ? x[r] + a.se.shift : x[r];
          av[4 * h + r] = y[r];
        }
      }
      if constexpr (MM == 0) settle_mfma();  // (the series branches on its degree)
      series_eval<MM>(m, u, w, a.se.e, lw);
      series_eval<DM>(m - 1, u, g, a.se.de, ld);
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int at = 32 * s + 16 * h + 4 * g4;
        const float4 rz = *(const float4*)(st + at), rg = *(const float4*)(st + kCh + at),
                     rm = *(const float4*)(st + 2 * kCh + at);
        const float z4[4] = {rz.x, rz.y, rz.z, rz.w}, g4_[4] = {rg.x, rg.y, rg.z, rg.w},
                    m4[4] = {rm.x, rm.y, rm.z, rm.w};
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          w[4 * h + r] *= z4[r];
          g[4 * h + r] *= fmaf(av[4 * h + r], g4_[r], m4[r]);
          if (kOwn && at + r < 16 * wave + l15) w[4 * h + r] = g[4 * h + r] = 0.f;
        }
      }
      // (an earlier query or gradient that is not finite times a masked zero is no
      // zero; without it, later ones still reach dk and dv, queries through w and
      // g, gradients through g and, column by column, at the end)
      const bool clean = kOwn && __ballot(bad);
      dirty |= clean;
      uint4 b[3];
      split3(w, b);
      contract<T, DT>(yb, s, l15, g4, b, sumv, clean);
      split3(g, b);
      contract<T, DT>(qb, s, l15, g4, b, sumk, clean);
    }
    add_chunk<L::kPl>(ck, dka[I]);
    add_chunk<L::kPl>(cv, dva[I]);
    if constexpr (flushes<T, DT>()) {
      if ((c - c_first) % kFlush == kFlush - 1) {
        const int row = (c_first + I) * kCh + 16 * wave + l15;
        const bool first = c - c_first == kFlush - 1;
        if (row < n) {
          flush_row((float*)a.dk + ((int64_t)head * n + row) * dk, dk, g4, dka[I], first);
          flush_row((float*)a.dv + ((int64_t)head * n + row) * dv, dv, g4, dva[I], first);
        }
      }
    }
  };
  if (c_first < nch) {
    fetch(c_first);
    put(c_first & 1, c_first);
    __syncthreads();
    for (int c = c_first; c < nch; ++c) {
      if (c + 1 < nch) fetch(c + 1);
      const u16* const base = smem16 + (c & 1) * L::kBuf;
      static_for<NQ>([&](auto ic) {
        constexpr int I = decltype(ic)::value;
        if (c > c_first + I) work(base, c, ic, std::false_type{});
        else if (c == c_first + I) work(base, c, ic, std::true_type{});
      });
      if (c + 1 < nch) put((c + 1) & 1, c + 1);
      __syncthreads();
    }
  }
#pragma unroll
  for (int i = 0; i < NQ; ++i) {
    const int row = (c_first + i) * kCh + 16 * wave + l15;
    if (row >= n) continue;
    if (dirty) {  // gradients of the own chunk that are not finite, for the keys at or before them
      for (int other = row; other < min(n, (c_first + i + 1) * kCh); ++other)
#pragma unroll
        for (int j = 0; j < DT; ++j)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int col = 16 * j + 4 * g4 + r;
            if (col < dv) dva[i][j][r] += sy.entry(other, col) * 0.f;
          }
    }
    [[maybe_unused]] const bool more = nch - c_first >= kFlush;
    store_row<T, DT>((T*)a.dk + ((int64_t)head * n + row) * dk, dk, g4, dka[i], 1.f, more);
    store_row<T, DT>((T*)a.dv + ((int64_t)head * n + row) * dv, dv, g4, dva[i], 1.f, more);
  }
}

template <typename T, int DT, int NQ, int PP>
hipError_t launch_pp(BwdArgs a, hipStream_t s) {
  using L = BwdLayout<T, DT>;
  static_assert(L::kBytes <= 160 * 1024, "LDS of one workgroup");
  auto rows = backward_rows<T, DT, NQ, PP>;
  auto cols = backward_cols<T, DT, NQ, PP>;
  if (L::kBytes > 64 * 1024) {
    for (const void* f : {(const void*)rows, (const void*)cols}) {
      hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, L::kBytes);
      if (e != hipSuccess) return e;
    }
  }
  a.blocks = (a.n + kCh * NQ - 1) / (kCh * NQ);
  a.by_xcd = a.heads >= 8;
  const unsigned grid = (unsigned)pair_blocks(a.heads, a.n, kCh * NQ);
  hipLaunchKernelGGL(rows, dim3(grid), dim3(kNW * 64), L::kBytes, s, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(cols, dim3(grid), dim3(kNW * 64), L::kBytes, s, a);
  return hipGetLastError();
}

// P = 4 has its series unrolled, the other orders share a kernel that loops over
// the coefficients (as in prefill_direct_kernel.hpp).
template <typename T, int DT>
hipError_t launch_dt(const BwdArgs& a, hipStream_t s) {
  if constexpr (sizeof(T) == 2) {
    if (backward_tiles(true, a.heads, a.n) == 2)
      return a.P == 4 ? launch_pp<T, DT, 2, 4>(a, s) : launch_pp<T, DT, 2, 0>(a, s);
  }
  return a.P == 4 ? launch_pp<T, DT, 1, 4>(a, s) : launch_pp<T, DT, 1, 0>(a, s);
}

template <typename T>
hipError_t launch_t(const BwdArgs& a, hipStream_t s) {
  switch ((std::max(a.dk_, a.dv_) + 15) / 16) {
    case 1: return launch_dt<T, 1>(a, s);
    case 2: return launch_dt<T, 2>(a, s);
    case 3: return launch_dt<T, 3>(a, s);
    default: return launch_dt<T, 4>(a, s);
  }
}

}  // namespace

size_t backward_direct_bytes(int BH, int n) {
  return sizeof(float) * (size_t)BH * (size_t)((n + kCh - 1) / kCh) * 3 * kCh;
}

hipError_t launch_backward_direct(const void* q, const void* k, const void* v, const void* dy, void* dq, void* dk,
                                  void* dv, bool bf16, int BH, int n, int dk_, int dv_, int P, float* stat,
                                  hipStream_t s) {
  BwdArgs a{q, k, v, dy, dq, dk, dv, stat, make_series(P, dk_), BH, n, dk_, dv_, P, 0, 0};
  return bf16 ? launch_t<u16>(a, s) : launch_t<float>(a, s);
}

}  // namespace sata
