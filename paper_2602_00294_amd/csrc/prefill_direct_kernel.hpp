// Causal prefill pair by pair: y_T = sum_{t<=T} w_Tt v_t / sum_{t<=T} w_Tt with
// w_Tt = f_P(q_T . k_t / sqrt(d_k)) (Sec. 2.1, the truncation of Sec. 2.4), on
// the matrix cores.  The sum over earlier tokens is the readout phi(q_T)^T S_T
// of the state form with the contraction over features carried out inside
// f_P, so the results are those of the chunked scan up to rounding.
//
// Work per head-token: (n / 2) 2 (d_k + d_v + 1) matrix flops against the
// scan's 2 D (d_v + 1) for the readout, and no features to generate.
//
// Bound: vector instructions.  Per 32 keys x 16 queries (P = 4, bfloat16) a wave
// issues 16 products of the series, 4 conversions and 2 + NCT matrix
// instructions, each of which keeps the vector unit from issuing for about 10
// cycles beside the 16 it runs.  Measured at B = 8, H = 32, n = 8192, d = 32:
// 1.45 ms (0.17 ps per pair, without a profiler) against 2.2 ms for the readout
// half of the scan; by the counters vector instructions issue on 73% of a
// SIMD's cycles and the matrix cores are busy on 43%, with 2.8 waves in flight.
// 1.90 ms before the chunks were read through buffer descriptors (no tests or
// 64-bit addresses per vector) and 2.37 ms with V transposed while staging.
// Two and four query tiles per wave took 1.54 and 1.53 ms (three: 1.48 in the
// same run).
//
// Layout.  The scores are computed transposed, S^T[key][query] = K Q^T, on
// v_mfma_f32_16x16x32_bf16: the result lane l holds query l % 16 and keys
// 4 (l / 16) .. +3 of a tile.  Two such tiles (32 keys) are, lane by lane, the
// B operand of O^T[column][query] += [V | 1]^T W^T with the K order "keys
// 4g .. 4g+3 of the first tile, then of the second" for lane group g = l / 16,
// so the weights never leave their lanes; V rows are read from LDS transposed,
// four keys of a column at a time (ds_read_b64_tr_b16), in that key order.
// The normaliser is the row of the constant-1 column of [V | 1].
//
// Split.  A workgroup of 4 waves owns 64 NQ queries of one head and walks the
// 64-token chunks of keys up to its last query.  Its 16-query tiles are dealt
// to the waves in turn (wave w: tiles w, w + 4, ...), so that each wave holds
// one tile of every 64-query chunk and the causal edge costs all four alike.
// K and V rows of a chunk are staged in LDS, double buffered, the next chunk
// fetched into registers meanwhile (a chunk is contiguous in memory: a thread's
// vectors lie at fixed offsets).
//
// Operands.  bfloat16 inputs: exact operands for the scores; weights of
// earlier chunks rounded to bfloat16, those of the query's own chunk carried
// as three bfloat16 numbers (24 bits).  float32 inputs: scores in float32
// (queries and keys as three bfloat16 numbers each, the six partial products
// of order 2^-16 and up: the series magnifies an error of the score by
// f'(|s|) / f(s), and hi + lo pairs left a row of d = 7, P = 6 1.1e-4 off);
// weights and values as hi + lo pairs with all four products (with three, as
// in the scan, y was a tenth further off than the scan's); and the query's own chunk in float32 on
// v_mfma_f32_16x16x4_f32.  At d_k <= 16 the 32 entries of a contraction step
// hold two numbers of each coordinate, so that the six products are three
// instructions: [kh|kl][ql|qh] + [kh|km][qm|qm] + [kh|km][qh|qh].
#pragma once

#include <hip/hip_runtime.h>

#include "kernels.hpp"
#include "route.hpp"
#include "series.hpp"

namespace sata {

namespace {

constexpr int kCh = 64;  // keys per staged chunk
constexpr int kNW = 4;   // waves per workgroup

// LDS map of one buffer: PL planes (hi, lo) of K rows [64][kKS], then of
// [V | 1] rows [64][kVR], bf16.  V rows start an odd multiple of 8 banks
// apart, so that the eight rows a half wave reads transposed lie in distinct
// banks.
template <bool X3, bool PK, int NKT, int NCT>
struct DirectLds {
  static constexpr int kPl = X3 ? 2 : 1;              // planes of V
  static constexpr int kPk = X3 ? (PK ? 2 : 3) : 1;  // planes of K
  static constexpr int kKS = 32 * NKT + 8;  // bf16 per key row (rows start 20 or 36 banks apart)
  static constexpr int kKPlane = kCh * kKS;
  static constexpr int kVR = 16 * (NCT | 1);
  static constexpr int kVPlane = kCh * kVR;
  static constexpr int kBuf = kPk * kKPlane + kPl * kVPlane;  // bf16 per buffer
  static constexpr int kBytes = 2 * kBuf * 2;
};

// T: input element (bf16 bits or float).  X3 (float inputs): split operands.
// PK (with X3, d_k <= 16): packed operands.  NKT: K steps of 32 covering d_k; NCT: column tiles of 16 covering d_v + 1;
// NQ: query tiles per wave.  nqb: workgroups per query head; heads: query
// heads, of which qg share one key/value head.  The grid is nqb * (heads
// rounded up to a multiple of 8) when by_xcd, else nqb * heads.
template <typename T, bool X3, bool PK, int NKT, int NCT, int NQ, int PP>
__global__ void __launch_bounds__(kNW * 64, (X3 ? NCT >= 4 || NKT == 2 : NCT >= 3 && NKT == 2) ? 2 : 3)
prefill_direct_kernel(const T* __restrict__ q_, const T* __restrict__ k_, const T* __restrict__ v_, T* __restrict__ y_,
                      Series se, int heads, int qg, int n, int dk, int dv, int P, int nqb, int by_xcd) {
  using L = DirectLds<X3, PK, NKT, NCT>;
  constexpr int kEV = 16 / sizeof(T);  // elements per 16-byte vector
  constexpr int KS = L::kKS;
  extern __shared__ __attribute__((aligned(16))) u16 smem16[];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int l15 = lane & 15;
  const int g4 = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // Workgroups go to the 8 XCDs in turn.  With 8 heads or more each XCD takes
  // whole heads, one after the other, so that a head's keys and values are
  // read through one L2; longest query blocks first.
  int qh, qb;
  if (by_xcd) {
    const int j = blockIdx.x >> 3;
    qh = (j / nqb) * 8 + (int)(blockIdx.x & 7);
    qb = nqb - 1 - j % nqb;
    if (qh >= heads) return;
  } else {
    qh = blockIdx.x % heads;
    qb = nqb - 1 - blockIdx.x / heads;
  }
  const int64_t kvh = qh / qg;
  const float coef = lane < kMaxSeries ? se.e[lane & (kMaxSeries - 1)] : 0.f;
  constexpr int MM = PP > 0 ? PP - 1 : 0;
  const T* const qp = q_ + (int64_t)qh * n * dk;
  const T* const kp = k_ + kvh * n * dk;
  const T* const vp = v_ + kvh * n * dv;
  T* const yp = y_ + (int64_t)qh * n * dv;
  const bool veck = dk % kEV == 0 && (((uintptr_t)qp | (uintptr_t)kp) & 15) == 0;
  const bool vecv = dv % kEV == 0 && ((uintptr_t)vp & 15) == 0;
  const int c_first = qb * NQ;                          // this workgroup's first query chunk
  const int chunks = min(c_first + NQ, (n + kCh - 1) / kCh);  // key chunks it walks

  // ---- the parts of both buffers that staging never writes: zero padding of
  // K rows past d_k; the constant-1 column of V rows and zeros past it
  for (int b = 0; b < 2; ++b) {
    u16* const kb = smem16 + b * L::kBuf;
    u16* const vb = kb + L::kPk * L::kKPlane;
    // (packed rows: two halves of 16 entries)
    const int padk = (PK ? 16 : 32 * NKT) - dk, padv = NCT * 16 - dv;
    for (int pl = 0; pl < L::kPk; ++pl)
      for (int h = 0; h < (PK ? 2 : 1); ++h)
        for (int i = tid; i < kCh * padk; i += kNW * 64)
          kb[pl * L::kKPlane + (i / padk) * KS + 16 * h + dk + i % padk] = 0;
    for (int pl = 0; pl < L::kPl; ++pl) {
      for (int i = tid; i < kCh * padv; i += kNW * 64)
        vb[pl * L::kVPlane + (i / padv) * L::kVR + dv + i % padv] = (i % padv == 0 && pl == 0) ? (u16)0x3f80 : (u16)0;
    }
  }

  // ---- this wave's queries: B operands of the scores, lane = query l15, in the
  // series' units
  constexpr int kQP = X3 ? 3 : 1;  // packed: [qh|qh], [qm|qm], [ql|qh]
  uint4 qf[NQ][NKT][kQP];
#pragma unroll
  for (int i = 0; i < NQ; ++i) {
    const int row = (c_first + i) * kCh + 16 * wave + l15;
#pragma unroll
    for (int kt = 0; kt < NKT; ++kt) {
      const int c0 = PK ? 8 * (g4 & 1) : 32 * kt + 8 * g4;
      if constexpr (X3) {
        float x[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) x[j] = row < n && c0 + j < dk ? qp[(int64_t)row * dk + c0 + j] * se.scale : 0.f;
#pragma unroll
        for (int pl = 0; pl < kQP; ++pl) {
          qf[i][kt][pl] = to_bf16(x);
          take_bf16(qf[i][kt][pl], x);
        }
        if (PK && g4 >= 2) qf[i][kt][kQP - 1] = qf[i][kt][0];
      } else {
        uint4 w = {0u, 0u, 0u, 0u};
        if (row < n) {
          if (veck) {
            if (c0 < dk) w = *(const uint4*)(qp + (int64_t)row * dk + c0);
          } else {
            uint32_t u[4] = {0u, 0u, 0u, 0u};
#pragma unroll
            for (int j = 0; j < 8; ++j)
              if (c0 + j < dk) u[j >> 1] |= (uint32_t)qp[(int64_t)row * dk + c0 + j] << (16 * (j & 1));
            w = uint4{u[0], u[1], u[2], u[3]};
          }
        }
        auto scaled = [&](uint32_t u) { return pack2(lo_f32(u) * se.scale, hi_f32(u) * se.scale); };
        qf[i][kt][0] = uint4{scaled(w.x), scaled(w.y), scaled(w.z), scaled(w.w)};
      }
    }
  }

  // ---- staging.  Rows of K and V as 16-byte vectors where the rows allow
  // them, else element by element; rows past the sequence are zero.
  constexpr int kItK = kCh * 32 * NKT / kEV / (kNW * 64);
  constexpr int kItV = (kCh * NCT * 16 / kEV + kNW * 64 - 1) / (kNW * 64);
  uint4 rk[kItK], rv[kItV];
  int ok[kItK], ov[kItV];         // where a vector goes in a plane (-1: past the rows)
  uint32_t sk[kItK], sv[kItV];    // where it comes from in a chunk
  const int nvk = dk / kEV, nvv = dv / kEV;  // vectors per row
#pragma unroll
  for (int i = 0; i < kItK; ++i) {
    const int idx = tid + i * kNW * 64;
    const bool on = veck && idx < kCh * nvk;
    ok[i] = on ? (idx / nvk) * KS + idx % nvk * kEV : -1;
    sk[i] = on ? 16u * idx : kNoVector;
  }
#pragma unroll
  for (int i = 0; i < kItV; ++i) {
    const int idx = tid + i * kNW * 64;
    const bool on = vecv && idx < kCh * nvv;
    ov[i] = on ? (idx / nvv) * L::kVR + idx % nvv * kEV : -1;
    sv[i] = on ? 16u * idx : kNoVector;
  }
  const VectorReader read_k(kp, (int64_t)n * dk * sizeof(T)), read_v(vp, (int64_t)n * dv * sizeof(T));
  // (chunks come in order, so the offsets move on by a chunk's bytes each time)
  auto fetch = [&]() {
#pragma unroll
    for (int i = 0; i < kItK; ++i) {
      rk[i] = read_k(sk[i]);
      sk[i] += kCh * dk * (int)sizeof(T);
    }
#pragma unroll
    for (int i = 0; i < kItV; ++i) {
      rv[i] = read_v(sv[i]);
      sv[i] += kCh * dv * (int)sizeof(T);
    }
  };
  // a vector into its row (float32: hi and lo planes)
  auto put_vec = [&](u16* dst, int plane, const uint4& w) {
    if constexpr (X3) {
      const float x[4] = {__uint_as_float(w.x), __uint_as_float(w.y), __uint_as_float(w.z), __uint_as_float(w.w)};
      const uint2 h = {pack2(x[0], x[1]), pack2(x[2], x[3])};
      *(uint2*)dst = h;
      *(uint2*)(dst + plane) = uint2{pack2(x[0] - lo_f32(h.x), x[1] - hi_f32(h.x)),
                                     pack2(x[2] - lo_f32(h.y), x[3] - hi_f32(h.y))};
    } else {
      *(uint4*)dst = w;
    }
  };
  // a vector of a float32 key row: its three numbers
  auto put_key = [&](u16* dst, const uint4& w) {
    float x[4] = {__uint_as_float(w.x), __uint_as_float(w.y), __uint_as_float(w.z), __uint_as_float(w.w)};
    uint2 p[3];
#pragma unroll
    for (int pl = 0; pl < 3; ++pl) {
      p[pl] = uint2{pack2(x[0], x[1]), pack2(x[2], x[3])};
      x[0] -= lo_f32(p[pl].x), x[1] -= hi_f32(p[pl].x), x[2] -= lo_f32(p[pl].y), x[3] -= hi_f32(p[pl].y);
    }
    *(uint2*)dst = p[0];
    if constexpr (PK) {
      *(uint2*)(dst + 16) = p[1];
      *(uint2*)(dst + L::kKPlane) = p[0];
      *(uint2*)(dst + L::kKPlane + 16) = p[2];
    } else {
      *(uint2*)(dst + L::kKPlane) = p[1];
      *(uint2*)(dst + 2 * L::kKPlane) = p[2];
    }
  };
  auto put_rows = [&](u16* dst, int stride, int plane, const T* src, int width, int c) {
    const int rows = min(kCh, n - c * kCh);
#pragma unroll 4
    for (int i = tid; i < kCh * width; i += kNW * 64) {
      const int row = i / width, at = row * stride + i - row * width;
      if constexpr (X3) {
        const float x = row < rows ? src[(int64_t)c * kCh * width + i] : 0.f;
        const uint32_t h = pack2(x, 0.f);
        dst[at] = (u16)h;
        dst[at + plane] = (u16)pack2(x - lo_f32(h), 0.f);
      } else {
        dst[at] = row < rows ? src[(int64_t)c * kCh * width + i] : (u16)0;
      }
    }
  };
  auto put = [&](int b, int c) {
    u16* const kb = smem16 + b * L::kBuf;
    u16* const vb = kb + L::kPk * L::kKPlane;
    if (veck) {
#pragma unroll
      for (int i = 0; i < kItK; ++i) {
        if (ok[i] < 0) continue;
        if constexpr (X3) put_key(kb + ok[i], rk[i]);
        else *(uint4*)(kb + ok[i]) = rk[i];
      }
    } else if constexpr (X3) {
      const int rows = min(kCh, n - c * kCh);
      for (int i = tid; i < kCh * dk; i += kNW * 64) {
        const int row = i / dk;
        float x = row < rows ? kp[(int64_t)c * kCh * dk + i] : 0.f;
        u16* const dst = kb + row * KS + i - row * dk;
        u16 p[3];
#pragma unroll
        for (int pl = 0; pl < 3; ++pl) {
          const uint32_t h = pack2(x, 0.f);
          p[pl] = (u16)h;
          x -= lo_f32(h);
        }
        dst[0] = p[0];
        if constexpr (PK) {
          dst[16] = p[1];
          dst[L::kKPlane] = p[0];
          dst[L::kKPlane + 16] = p[2];
        } else {
          dst[L::kKPlane] = p[1];
          dst[2 * L::kKPlane] = p[2];
        }
      }
    } else {
      put_rows(kb, KS, L::kKPlane, kp, dk, c);
    }
    if (vecv) {
#pragma unroll
      for (int i = 0; i < kItV; ++i)
        if (ov[i] >= 0) put_vec(vb + ov[i], L::kVPlane, rv[i]);
    } else {
      put_rows(vb, L::kVR, L::kVPlane, vp, dv, c);
    }
  };
  // V^T operand of column tile j for keys 32 s .. +31: two transposed reads of
  // four keys; lane l of each 16 reads row l / 4, columns 4 (l % 4) .. +3
  const int vt_at = (4 * g4 + (l15 >> 2)) * L::kVR + 4 * (l15 & 3);
  auto load_vt = [&](const u16* vb, int s, int j) {
    return read_transposed(vb + vt_at + 32 * s * L::kVR + 16 * j, 16 * L::kVR);
  };

  f32x4 O[NQ][NCT];
#pragma unroll
  for (int i = 0; i < NQ; ++i)
#pragma unroll
    for (int j = 0; j < NCT; ++j) O[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  // A operands of keys 32 s + 16 h .. +15
  auto load_keys = [&](const u16* kb, int s, int h, uint4 (&ka)[NKT][L::kPk]) {
#pragma unroll
    for (int kt = 0; kt < NKT; ++kt)
#pragma unroll
      for (int pl = 0; pl < L::kPk; ++pl)
        ka[kt][pl] = *(const uint4*)(kb + pl * L::kKPlane + (32 * s + 16 * h + l15) * KS + 32 * kt + 8 * g4);
  };
  // u = score + sqrt(d_k), in the series' units, of query tile i against 16 keys
  // (smallest products first)
  auto scores = [&](const uint4 (&ka)[NKT][L::kPk], int i, float* u) {
    f32x4 a = {se.shift, se.shift, se.shift, se.shift};
#pragma unroll
    for (int kt = 0; kt < NKT; ++kt) {
      if constexpr (PK) {
        a = mfma_bf16(ka[kt][1], qf[i][kt][2], a);
        a = mfma_bf16(ka[kt][0], qf[i][kt][1], a);
        a = mfma_bf16(ka[kt][0], qf[i][kt][0], a);
      } else {
#pragma unroll
        for (int t = 2; t >= 0; --t)
#pragma unroll
          for (int x = 0; x <= t; ++x)
            if (x < L::kPk && t - x < kQP) a = mfma_bf16(ka[kt][x], qf[i][kt][t - x], a);
      }
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) u[r] = a[r];
  };
  // one 32-key step for the query tiles I0 .. NQ - 1 (all of whose keys are in
  // earlier chunks)
  auto full_step = [&](const u16* kb, const u16* vb, int s, auto i0c) {
    constexpr int I0 = decltype(i0c)::value, M = NQ - I0;
    float x[8 * M], w[8 * M];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      uint4 ka[NKT][L::kPk];
      load_keys(kb, s, h, ka);
#pragma unroll
      for (int i = 0; i < M; ++i) scores(ka, I0 + i, x + 8 * i + 4 * h);
    }
    series_eval<MM>(P - 1, x, w, se.e, coef);
    uint4 b[M], bl[X3 ? M : 1];
#pragma unroll
    for (int i = 0; i < M; ++i) {
      b[i] = to_bf16(w + 8 * i);
      if constexpr (X3) {
        take_bf16(b[i], w + 8 * i);
        bl[i] = to_bf16(w + 8 * i);
      }
    }
#pragma unroll
    for (int j = 0; j < NCT; ++j) {
      const uint4 va = load_vt(vb, s, j);
      uint4 vl;
      if constexpr (X3) vl = load_vt(vb + L::kVPlane, s, j);
#pragma unroll
      for (int i = 0; i < M; ++i) {
        if constexpr (X3) {
          O[I0 + i][j] = mfma_bf16(vl, bl[i], O[I0 + i][j]);
          O[I0 + i][j] = mfma_bf16(va, bl[i], O[I0 + i][j]);
          O[I0 + i][j] = mfma_bf16(vl, b[i], O[I0 + i][j]);
        }
        O[I0 + i][j] = mfma_bf16(va, b[i], O[I0 + i][j]);
      }
    }
  };
  // query tile i against its own chunk c (tokens up to the query)
  auto own_chunk = [&](const u16* kb, const u16* vb, int i, int c) {
    if constexpr (X3) {
      // float32 products, operands straight from memory (each is read once)
      const int row = c * kCh + 16 * wave + l15;
      for (int kt = 0; kt <= wave; ++kt) {
        const int key = c * kCh + 16 * kt + l15;
        f32x4 a = {se.shift, se.shift, se.shift, se.shift};
        for (int kk = 0; kk < dk; kk += 4) {
          const int col = kk + g4;
          const float xk = (key < n && col < dk) ? (float)kp[(int64_t)key * dk + col] : 0.f;
          const float xq = (row < n && col < dk) ? (float)qp[(int64_t)row * dk + col] * se.scale : 0.f;
          a = mfma_f32(xk, xq, a);
        }
        float x[4], w[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) x[r] = a[r];
        series_eval<MM>(P - 1, x, w, se.e, coef);
        if (kt == wave) {
#pragma unroll
          for (int r = 0; r < 4; ++r)
            if (4 * g4 + r > l15) w[r] = 0.f;
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int kr = c * kCh + 16 * kt + 4 * g4 + r;
#pragma unroll
          for (int j = 0; j < NCT; ++j) {
            const int col = 16 * j + l15;
            const float xv = (kr < n && col < dv) ? (float)vp[(int64_t)kr * dv + col] : (col == dv ? 1.f : 0.f);
            O[i][j] = mfma_f32(xv, w[r], O[i][j]);
          }
        }
      }
    } else {
      for (int s = 0; s <= (wave >> 1); ++s) {
        float x[8], w[8];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          uint4 ka[NKT][L::kPk];
          load_keys(kb, s, h, ka);
          scores(ka, i, x + 4 * h);
        }
        series_eval<MM>(P - 1, x, w, se.e, coef);
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int r = 0; r < 4; ++r)
            if (32 * s + 16 * h + 4 * g4 + r > 16 * wave + l15) w[4 * h + r] = 0.f;
        const uint4 b0 = to_bf16(w);
        take_bf16(b0, w);
        const uint4 b1 = to_bf16(w);
        take_bf16(b1, w);
        const uint4 b2 = to_bf16(w);
#pragma unroll
        for (int j = 0; j < NCT; ++j) {
          uint4 va = load_vt(vb, s, j);
          // (a step's second 16 keys are all masked for the tile of its first 16
          // queries; a value there that is not finite would not be zero times 0)
          if (2 * s == wave) va.z = va.w = 0u;
          O[i][j] = mfma_bf16(va, b2, O[i][j]);
          O[i][j] = mfma_bf16(va, b1, O[i][j]);
          O[i][j] = mfma_bf16(va, b0, O[i][j]);
        }
      }
    }
  };

  fetch();
  put(0, 0);
  __syncthreads();
  for (int c = 0; c < chunks; ++c) {
    if (c + 1 < chunks) fetch();
    const u16* const kb = smem16 + (c & 1) * L::kBuf;
    const u16* const vb = kb + L::kPk * L::kKPlane;
    if (c < c_first) {
      full_step(kb, vb, 0, std::integral_constant<int, 0>{});
      full_step(kb, vb, 1, std::integral_constant<int, 0>{});
    } else {
      static_for<NQ>([&](auto ic) {
        constexpr int I = decltype(ic)::value;
        if (c_first + I == c) {
          own_chunk(kb, vb, I, c);
          if constexpr (I + 1 < NQ) {
            full_step(kb, vb, 0, std::integral_constant<int, I + 1>{});
            full_step(kb, vb, 1, std::integral_constant<int, I + 1>{});
          }
        }
      });
    }
    // the other buffer was last read before the previous barrier
    if (c + 1 < chunks) put((c + 1) & 1, c + 1);
    __syncthreads();
  }

  // ---- y = O / normaliser: lane holds columns 16 j + 4 g4 .. +3 of query l15;
  // the normaliser sits in the lane group that holds column d_v
  const int jn = dv >> 4, gn = (dv >> 2) & 3, rn = dv & 3;
  const bool vecy = dv % 4 == 0 && ((uintptr_t)yp & (4 * sizeof(T) - 1)) == 0;
#pragma unroll
  for (int i = 0; i < NQ; ++i) {
    const int row = (c_first + i) * kCh + 16 * wave + l15;
    float z = 0.f;
#pragma unroll
    for (int j = 0; j < NCT; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (j == jn && r == rn) z = O[i][j][r];
    z = __shfl(z, 16 * gn + l15);
    if (row >= n) continue;
#pragma unroll
    for (int j = 0; j < NCT; ++j) {
      const int c0 = 16 * j + 4 * g4;
      float o[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) o[r] = O[i][j][r] / z;
      T* const p = yp + (int64_t)row * dv + c0;
      if (vecy) {
        if (c0 < dv) {
          if constexpr (std::is_same_v<T, float>) {
            *(float4*)p = float4{o[0], o[1], o[2], o[3]};
          } else {
            *(uint2*)p = uint2{(uint32_t)f32_to_bf16(o[0]).bits | ((uint32_t)f32_to_bf16(o[1]).bits << 16),
                               (uint32_t)f32_to_bf16(o[2]).bits | ((uint32_t)f32_to_bf16(o[3]).bits << 16)};
          }
        }
      } else {
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (c0 + r < dv) {
            if constexpr (std::is_same_v<T, float>) p[r] = o[r];
            else p[r] = f32_to_bf16(o[r]).bits;
          }
      }
    }
  }
}

template <typename T, bool X3, bool PK, int NKT, int NCT, int NQ, int PP>
hipError_t launch_p(const void* q, const void* k, const void* v, void* y, int heads, int qg, int n, int dk, int dv,
                      int P, hipStream_t s) {
  constexpr int bytes = DirectLds<X3, PK, NKT, NCT>::kBytes;
  static_assert(bytes <= 160 * 1024, "LDS of one workgroup");
  auto kern = prefill_direct_kernel<T, X3, PK, NKT, NCT, NQ, PP>;
  if (bytes > 64 * 1024) {
    hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    if (e != hipSuccess) return e;
  }
  const Series se = make_series(P, dk);
  const int nqb = (n + kCh * NQ - 1) / (kCh * NQ);
  const int by_xcd = heads >= 8;
  const unsigned grid = (unsigned)pair_blocks(heads, n, kCh * NQ);
  hipLaunchKernelGGL(kern, dim3(grid), dim3(kNW * 64), bytes, s, (const T*)q, (const T*)k, (const T*)v, (T*)y, se,
                     heads, qg, n, dk, dv, P, nqb, by_xcd);
  return hipGetLastError();
}

// P = 4, the order of the benchmark's workloads, has its series unrolled; the
// other orders share one kernel that reads the coefficients from a lane in a
// loop.  Measured (128 heads, n = 8192, ps per pair, whole call): d = 16
// bfloat16 P = 2, 3 by the loop 0.109, 0.144, P = 4 unrolled 0.146; float32
// 0.403, 0.415, 0.401.  So unrolling is worth about a term of the series (0.03
// to 0.06 ps); an unrolled kernel for each order would be 3.5 times the compiled
// kernels for that.
template <typename T, bool X3, bool PK, int NKT, int NCT, int NQ>
hipError_t launch_one(const void* q, const void* k, const void* v, void* y, int heads, int qg, int n, int dk, int dv,
                      int P, hipStream_t s) {
  return P == 4 ? launch_p<T, X3, PK, NKT, NCT, NQ, 4>(q, k, v, y, heads, qg, n, dk, dv, P, s)
                : launch_p<T, X3, PK, NKT, NCT, NQ, 0>(q, k, v, y, heads, qg, n, dk, dv, P, s);
}

template <typename T, bool X3, bool PK, int NKT, int NCT>
hipError_t launch_nq(const void* q, const void* k, const void* v, void* y, int heads, int qg, int n, int dk, int dv,
                     int P, hipStream_t s) {
  constexpr int kWide = direct_wide_tiles(X3, NCT);
  if (direct_query_tiles(X3, dv, heads, n) == kWide)
    return launch_one<T, X3, PK, NKT, NCT, kWide>(q, k, v, y, heads, qg, n, dk, dv, P, s);
  return launch_one<T, X3, PK, NKT, NCT, 1>(q, k, v, y, heads, qg, n, dk, dv, P, s);
}

template <typename T, bool X3, bool PK, int NKT>
hipError_t launch_nct(const void* q, const void* k, const void* v, void* y, int heads, int qg, int n, int dk, int dv,
                      int P, hipStream_t s) {
  switch ((dv + 16) / 16) {
    case 1: return launch_nq<T, X3, PK, NKT, 1>(q, k, v, y, heads, qg, n, dk, dv, P, s);
    case 2: return launch_nq<T, X3, PK, NKT, 2>(q, k, v, y, heads, qg, n, dk, dv, P, s);
    case 3: return launch_nq<T, X3, PK, NKT, 3>(q, k, v, y, heads, qg, n, dk, dv, P, s);
    case 4: return launch_nq<T, X3, PK, NKT, 4>(q, k, v, y, heads, qg, n, dk, dv, P, s);
    default: return launch_nq<T, X3, PK, NKT, 5>(q, k, v, y, heads, qg, n, dk, dv, P, s);
  }
}

}  // namespace

}  // namespace sata
