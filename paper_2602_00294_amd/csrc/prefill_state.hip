// The state after a sequence, S = sum_t phi(k_t) (x) [v_t, 1] (App. A2, the
// accumulated feature states), as one contraction over the tokens on
// v_mfma_f32_16x16x32_bf16 with float32 accumulators.  It serves the prefills
// whose outputs are computed pair by pair (prefill_direct.hip), which need the
// states of no token but the last.
//
// A feature is a product (smallest symbol i1) x (tuple g of the rest)
// (state_table.hpp).  A wave owns a block of GT tiles of 16 tuples g times IT
// multipliers i1 and keeps its GT * IT * NCT accumulator tiles in registers
// for the whole sequence.  Per 32 tokens it forms phi_g of its tiles in
// float32 (lane l: tuple l % 16, tokens 8 (l / 16) .. +7: the A operand's own
// layout, read from coordinate rows in LDS), and for each i1 multiplies by
// k[i1], rounds once to bfloat16 (float32 inputs: hi + lo pairs, three
// products) and contracts with [V | 1].  Nothing but the coordinates and V
// passes through LDS, and the weights enter once, at the end.
//
// Bound: no one unit alone.  Forming 512 feature-tokens takes 8 products and 4
// conversions beside NCT matrix instructions; with phi_g, staging, normalisers
// and padded slots the counters show 19 vector and 2.5 matrix instructions
// (B = 8, H = 32, n = 8192, d = 32, P = 4 bfloat16), vector issue on 55% of a
// SIMD's cycles (51% at d = 64), matrix cores busy on 25%, and 1.7 waves in
// flight of the 2 that the registers leave: chunks end at a barrier and
// workgroups are uneven.  Times, with those before the table entries and
// weights were fetched ahead of the stores: 1.99 ms (2.14), 0.95 ns per
// head-token (the update half of the scan: 2.2 ms); B = 64, H = 32, n = 2048,
// d = 16: 0.89 ms (0.99); B = 2, H = 8, n = 4096, d = 64: 0.58 ms (0.76; the
// whole scan 3.8).  Tiles one after the other with their multipliers in
// registers took 2.13 ms where rows of tiles per multiplier took 2.42.
//
// Normaliser.  A column of its own for the constant 1 would cost a whole
// column tile when d_v is a multiple of 16.  There, blocks of their own take
// phi_g contracted with the keys: sum_t phi_g(k_t) k_t[i1] is the normaliser
// of (i1, g), 16 multipliers a product.
//
// Workgroups of 4 waves share the staged tokens (64 at a time, double
// buffered, the next ones fetched into registers meanwhile).  Where blocks
// times heads leave the chip idle the tokens are cut into parts, whose sums a
// second kernel adds in part order.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>

#include "kernels.hpp"
#include "series.hpp"
#include "state_table.hpp"

namespace sata {

namespace {

constexpr int kCh = 64;       // tokens per staged chunk
constexpr int kNW = 4;        // waves per workgroup
constexpr int kRS = kCh + 4;  // floats per coordinate row (rows start 4 banks apart)

__device__ __forceinline__ uint4 rest_bf16(const float (&x)[8], const uint4& h) {
  return uint4{pack2(x[0] - lo_f32(h.x), x[1] - hi_f32(h.x)), pack2(x[2] - lo_f32(h.y), x[3] - hi_f32(h.y)),
               pack2(x[4] - lo_f32(h.z), x[5] - hi_f32(h.z)), pack2(x[6] - lo_f32(h.w), x[7] - hi_f32(h.w))};
}
__device__ __forceinline__ void load8(const float* p, float (&x)[8]) {
  const float4 a = *(const float4*)p, b = *(const float4*)(p + 4);
  x[0] = a.x, x[1] = a.y, x[2] = a.z, x[3] = a.w, x[4] = b.x, x[5] = b.y, x[6] = b.z, x[7] = b.w;
}

// bf16 per LDS row of [V | 1]: an odd multiple of 8 banks, so that the rows a
// half wave reads transposed lie in distinct banks.
__host__ __device__ constexpr int v_row(int nct) { return 16 * (nct | 1); }

struct StateArgs {
  const uint64_t* gsym;
  const StateBlock* list;
  const int32_t* ftab;
  const int32_t* ztab;
  const float* weight;
  float* out;  // [parts][BH][D][d_v + 1]
  int64_t D;
  int BH, n, dk, dv;
  int part_len;  // tokens per part (multiple of 64)
  int nwg;       // workgroups per head
  int lwg, zwg;  // the first workgroups of low blocks and of normaliser blocks
  int zcols;
  int mg;      // symbols per tuple g
  int by_xcd;  // grid.x = nwg * heads rounded up to 8, each XCD taking whole heads
  int ones;    // the constant-1 column is column d_v of [V | 1]
};

// T: input element (bf16 bits or float); X3 (float): split operands; NCT:
// column tiles; MG: symbols per tuple g (0: args.mg, any number).
template <typename T, bool X3, int NCT, int MG>
__global__ void __launch_bounds__(kNW * 64, 2) prefill_state_kernel(const T* __restrict__ k_, const T* __restrict__ v_,
                                                                    StateArgs a) {
  constexpr int GT = state_gt(NCT, X3), IT = state_it(NCT, X3);
  constexpr int PL = X3 ? 2 : 1;
  constexpr int kEV = 16 / sizeof(T);
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int dk = a.dk, dv = a.dv, n = a.n;
  // one buffer: coordinate rows of the d_k + 1 symbols (float32; the last holds
  // ones), then PL planes of [V | 1] rows
  constexpr int VR = v_row(NCT), kVPlane = kCh * VR;
  const int kt_bytes = (dk + 1) * kRS * 4;
  const int buf_bytes = kt_bytes + PL * kVPlane * 2;
  const int tid = threadIdx.x, lane = tid & 63, l15 = lane & 15, g4 = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int bh, wg;
  if (a.by_xcd) {
    const int j = blockIdx.x >> 3;
    bh = (j / a.nwg) * 8 + (int)(blockIdx.x & 7);
    wg = j % a.nwg;
    if (bh >= a.BH) return;
  } else {
    bh = blockIdx.x % a.BH;
    wg = blockIdx.x / a.BH;
  }
  const bool zwg = wg >= a.zwg;  // (uniform over the workgroup)
  const StateBlock blk = a.list[wg * kNW + wave];
  const bool live = blk.g0 >= 0;
  const T* const kp = k_ + (int64_t)bh * n * dk;
  const T* const vp = v_ + (int64_t)bh * n * dv;
  const int t_begin = blockIdx.y * a.part_len, t_end = min(n, t_begin + a.part_len);
  const bool veck = dk % 2 == 0 && ((uintptr_t)kp & (2 * sizeof(T) - 1)) == 0;
  const bool vecv = dv % kEV == 0 && ((uintptr_t)vp & 15) == 0;

  // ---- what staging never writes: the row of ones (cut at the part's end in
  // its last chunk), the constant-1 column of V rows and zeros past it
  for (int b = 0; b < 2; ++b) {
    if (tid < kRS) ((float*)(smem + b * buf_bytes))[dk * kRS + tid] = 1.f;
    u16* const vb = (u16*)(smem + b * buf_bytes + kt_bytes);
    const int pad = NCT * 16 - dv;
    for (int pl = 0; pl < PL; ++pl)
      for (int i = tid; i < kCh * pad; i += kNW * 64)
        vb[pl * kVPlane + (i / pad) * VR + dv + i % pad] = (i % pad == 0 && a.ones && pl == 0) ? (u16)0x3f80 : (u16)0;
  }

  // ---- this lane's tuples: where the coordinate rows of their symbols start
  // (more than two symbols a tuple: the packed symbols).  A normaliser block
  // has fewer tiles than a feature block, and the last one's end with the list.
  const int gts = zwg ? state_zt(X3) : GT;
  constexpr int kOff = MG ? MG : 1;
  int off[GT][kOff];
  uint64_t gs[MG ? 1 : GT];
#pragma unroll
  for (int t = 0; t < GT; ++t) {
    const uint64_t w = live && t < gts ? a.gsym[(blk.g0 + t) * 16 + l15] : 0;
#pragma unroll
    for (int j = 0; j < kOff; ++j) off[t][j] = (int)((w >> (8 * j)) & 0xff) * kRS + 8 * g4;
    if constexpr (MG == 0) gs[t] = w;
  }

  // ---- staging.  K transposed: an item is 4 tokens x 2 coordinates (two
  // float4 into coordinate rows); V as 16-byte vectors of its rows; element by
  // element where the rows do not allow either.  Tokens past the end are zero.
  constexpr int kItK = 2;  // 16 token quads x d_k / 2 pairs <= 512 items
  constexpr int kItV = (kCh * NCT * 16 / kEV + kNW * 64 - 1) / (kNW * 64);
  using Pair = std::conditional_t<X3, float2, uint32_t>;
  Pair rk[kItK][4];
  uint4 rv[kItV];
  const int pairs = dk / 2, nvv = dv / kEV;
  const VectorReader read_k(kp, (int64_t)t_end * dk * sizeof(T)), read_v(vp, (int64_t)t_end * dv * sizeof(T));
  uint32_t ks_at[kItK], sv[kItV];  // where an item comes from (kNoVector on: nowhere)
  int kd_at[kItK], ov[kItV];       // where it goes in a buffer (-1: nowhere)
#pragma unroll
  for (int i = 0; i < kItK; ++i) {
    const int idx = tid + i * kNW * 64;
    const int tq = idx / max(pairs, 1), cp = idx - tq * pairs;
    const bool on = veck && idx < kCh / 4 * pairs;
    ks_at[i] = on ? (uint32_t)((t_begin + 4 * tq) * dk + 2 * cp) * (int)sizeof(T) : kNoVector;
    kd_at[i] = on ? 2 * cp * kRS + 4 * tq : -1;
  }
#pragma unroll
  for (int i = 0; i < kItV; ++i) {
    const int idx = tid + i * kNW * 64;
    const bool on = vecv && idx < kCh * nvv;
    ov[i] = on ? (idx / nvv) * VR + idx % nvv * kEV : -1;
    sv[i] = on ? (uint32_t)t_begin * dv * (int)sizeof(T) + 16u * idx : kNoVector;
  }
  // (chunks come in order, so the offsets move on by a chunk's bytes each time)
  auto fetch = [&]() {
#pragma unroll
    for (int i = 0; i < kItK; ++i) {
      if (i > 0 && pairs <= 16) break;  // (one item a thread)
#pragma unroll
      for (int u = 0; u < 4; ++u) rk[i][u] = read_k.part<Pair>(ks_at[i] + u * dk * (int)sizeof(T));
      ks_at[i] += kCh * dk * (int)sizeof(T);
    }
#pragma unroll
    for (int i = 0; i < kItV; ++i) {
      rv[i] = read_v(sv[i]);
      sv[i] += kCh * dv * (int)sizeof(T);
    }
  };
  auto first = [](const Pair& p) -> float {
    if constexpr (X3) return p.x;
    else return lo_f32(p);
  };
  auto second = [](const Pair& p) -> float {
    if constexpr (X3) return p.y;
    else return hi_f32(p);
  };
  auto put = [&](int b, int t0) {
    float* const kt = (float*)(smem + b * buf_bytes);
    u16* const vb = (u16*)(smem + b * buf_bytes + kt_bytes);
    const int rows = t_end - t0;
    if (veck) {
#pragma unroll
      for (int i = 0; i < kItK; ++i) {
        if (i > 0 && pairs <= 16) break;
        if (kd_at[i] < 0) continue;
        *(float4*)(kt + kd_at[i]) = float4{first(rk[i][0]), first(rk[i][1]), first(rk[i][2]), first(rk[i][3])};
        *(float4*)(kt + kd_at[i] + kRS) = float4{second(rk[i][0]), second(rk[i][1]), second(rk[i][2]), second(rk[i][3])};
      }
    } else {
#pragma unroll 4
      for (int i = tid; i < kCh * dk; i += kNW * 64) {
        const int t = i / dk, c = i - t * dk;
        float x = 0.f;
        if (t < rows) {
          if constexpr (X3) x = kp[(int64_t)t0 * dk + i];
          else x = __uint_as_float((uint32_t)kp[(int64_t)t0 * dk + i] << 16);
        }
        kt[c * kRS + t] = x;
      }
    }
    if (vecv) {
#pragma unroll
      for (int i = 0; i < kItV; ++i) {
        if (ov[i] < 0) continue;
        if constexpr (X3) {
          const uint4 w = rv[i];
          const float x[4] = {__uint_as_float(w.x), __uint_as_float(w.y), __uint_as_float(w.z), __uint_as_float(w.w)};
          const uint2 h = {pack2(x[0], x[1]), pack2(x[2], x[3])};
          *(uint2*)(vb + ov[i]) = h;
          *(uint2*)(vb + ov[i] + kVPlane) = uint2{pack2(x[0] - lo_f32(h.x), x[1] - hi_f32(h.x)),
                                                  pack2(x[2] - lo_f32(h.y), x[3] - hi_f32(h.y))};
        } else {
          *(uint4*)(vb + ov[i]) = rv[i];
        }
      }
    } else {
#pragma unroll 4
      for (int i = tid; i < kCh * dv; i += kNW * 64) {
        const int t = i / dv, at = t * VR + i - t * dv;
        if constexpr (X3) {
          const float x = t < rows ? vp[(int64_t)t0 * dv + i] : 0.f;
          const uint32_t h = pack2(x, 0.f);
          vb[at] = (u16)h;
          vb[at + kVPlane] = (u16)pack2(x - lo_f32(h), 0.f);
        } else {
          vb[at] = t < rows ? vp[(int64_t)t0 * dv + i] : (u16)0;
        }
      }
    }
    // every monomial of a token past the end is zero
    if (rows < kCh && tid < kCh) kt[dk * kRS + tid] = tid < rows ? 1.f : 0.f;
  };
  // B operand of column tile j for tokens 32 s .. +31 (lane: column l15, tokens
  // 8 g4 .. +7): two transposed reads of four tokens
  const int vt_at = (8 * g4 + (l15 >> 2)) * VR + 4 * (l15 & 3);
  auto load_vt = [&](const u16* vb, int s, int j) {
    return read_transposed(vb + vt_at + 32 * s * VR + 16 * j, 4 * VR);
  };

  // phi_g (without weights) of tile t for tokens 32 s + 8 g4 .. +7
  auto make_g = [&](const float* kt, int s, int t, float (&gv)[8]) {
    load8(kt + off[t][0] + 32 * s, gv);
    if constexpr (MG > 1) {
#pragma unroll
      for (int j = 1; j < MG; ++j) {
        float x[8];
        load8(kt + off[t][j] + 32 * s, x);
#pragma unroll
        for (int e = 0; e < 8; ++e) gv[e] *= x[e];
      }
    }
    if constexpr (MG == 0)
      for (int j = 1; j < a.mg; ++j) {
        float x[8];
        load8(kt + (int)((gs[t] >> (8 * j)) & 0xff) * kRS + 8 * g4 + 32 * s, x);
#pragma unroll
        for (int e = 0; e < 8; ++e) gv[e] *= x[e];
      }
  };

  // every chunk of the part through LDS: work(coordinate rows, V rows)
  auto each_chunk = [&](auto&& work) {
    if (t_begin >= t_end) return;
    fetch();
    __syncthreads();  // the constant rows are written before the first chunk's may change them
    put(0, t_begin);
    __syncthreads();
    int b = 0;
    for (int t0 = t_begin; t0 < t_end; t0 += kCh, b ^= 1) {
      const bool more = t0 + kCh < t_end;
      if (more) fetch();
      const char* const base = smem + b * buf_bytes;
      if (live) work((const float*)base, (const u16*)(base + kt_bytes));
      if (more) put(b ^ 1, t0 + kCh);  // (last read before the previous barrier)
      __syncthreads();
    }
  };
  const int E = dv + 1;
  float* const out = a.out + ((int64_t)blockIdx.y * a.BH + bh) * a.D * E;

  // ---- a normaliser block: phi_g of its tiles times KT tiles of the keys
  auto normaliser_block = [&](auto ktc) {
    constexpr int KT = decltype(ktc)::value, ZT = state_zt(X3);
    static_assert(ZT <= GT, "symbols of a normaliser block's tiles");
    f32x4 acc[ZT][KT];
#pragma unroll
    for (int t = 0; t < ZT; ++t)
#pragma unroll
      for (int z = 0; z < KT; ++z) acc[t][z] = f32x4{0.f, 0.f, 0.f, 0.f};
    // (multipliers past d_k repeat the row of ones; they are not stored)
    int zrow[KT];
#pragma unroll
    for (int z = 0; z < KT; ++z) zrow[z] = min(16 * z + l15, dk) * kRS + 8 * g4;
    each_chunk([&](const float* kt, const u16*) {
      f32x4 d[X3 ? ZT : 1][X3 ? KT : 1];
      if constexpr (X3) {
#pragma unroll
        for (int t = 0; t < ZT; ++t)
#pragma unroll
          for (int z = 0; z < KT; ++z) d[t][z] = f32x4{0.f, 0.f, 0.f, 0.f};
      }
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        uint4 h[ZT], l[X3 ? ZT : 1];
#pragma unroll
        for (int t = 0; t < ZT; ++t) {
          float gv[8];
          make_g(kt, s, t, gv);
          h[t] = to_bf16(gv);
          if constexpr (X3) l[t] = rest_bf16(gv, h[t]);
        }
#pragma unroll
        for (int z = 0; z < KT; ++z) {
          float x[8];
          load8(kt + zrow[z] + 32 * s, x);
          const uint4 kh = to_bf16(x);
          if constexpr (X3) {
            // (the keys in three numbers: these sums take the same rounding,
            // that of phi_g alone, as a column of ones would)
            take_bf16(kh, x);
            const uint4 km = to_bf16(x);
            take_bf16(km, x);
            const uint4 kl = to_bf16(x);
#pragma unroll
            for (int t = 0; t < ZT; ++t) {
              d[t][z] = mfma_bf16(l[t], km, mfma_bf16(h[t], kl, d[t][z]));
              d[t][z] = mfma_bf16(l[t], kh, mfma_bf16(h[t], km, d[t][z]));
              d[t][z] = mfma_bf16(h[t], kh, d[t][z]);
            }
          } else {
#pragma unroll
            for (int t = 0; t < ZT; ++t) acc[t][z] = mfma_bf16(h[t], kh, acc[t][z]);
          }
        }
      }
      if constexpr (X3) {
#pragma unroll
        for (int t = 0; t < ZT; ++t)
#pragma unroll
          for (int z = 0; z < KT; ++z) acc[t][z] += d[t][z];
      }
    });
    if (!live) return;
    // a tile's table entries one tile ahead, its weights together
    int f[2][KT][4];
    auto entries = [&](int t, int (&to)[KT][4]) {
#pragma unroll
      for (int z = 0; z < KT; ++z)
#pragma unroll
        for (int r_ = 0; r_ < 4; ++r_)
          to[z][r_] = 16 * z < a.zcols
                          ? a.ztab[(int64_t)((blk.g0 + t) * 16 + 4 * g4 + r_) * a.zcols + 16 * z + l15]
                          : -1;
    };
    entries(0, f[0]);
#pragma unroll
    for (int t = 0; t < ZT; ++t) {
      const int(&ft)[KT][4] = f[t & 1];
      float w[KT][4];
#pragma unroll
      for (int z = 0; z < KT; ++z)
#pragma unroll
        for (int r_ = 0; r_ < 4; ++r_) w[z][r_] = a.weight[max(ft[z][r_], 0)];
      if (t + 1 < ZT) entries(t + 1, f[(t + 1) & 1]);
#pragma unroll
      for (int z = 0; z < KT; ++z)
#pragma unroll
        for (int r_ = 0; r_ < 4; ++r_)
          if (ft[z][r_] >= 0) out[(int64_t)ft[z][r_] * E + dv] = acc[t][z][r_] * w[z][r_];
    }
  };
  if (zwg) {
    if (a.zcols <= 48) normaliser_block(std::integral_constant<int, 3>{});
    else normaliser_block(std::integral_constant<int, 5>{});
    return;
  }

  // ---- a block of features: R rows (multipliers) of up to GT tiles.  Tiles
  // one after the other, the next one's coordinates on their way meanwhile;
  // the multipliers of a step stay in registers.
  auto feature_block = [&](auto rc) {
    constexpr int R = decltype(rc)::value;
    f32x4 acc[GT][R][NCT];
#pragma unroll
    for (int t = 0; t < GT; ++t)
#pragma unroll
      for (int i = 0; i < R; ++i)
#pragma unroll
        for (int j = 0; j < NCT; ++j) acc[t][i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    each_chunk([&](const float* kt, const u16* vt) {
      // (the tile count is read afresh each time so that its tests are not
      // held in registers)
      int tiles = blk.tiles;
      asm volatile("" : "+s"(tiles));
      const float* const mr = kt + blk.i0 * kRS + 8 * g4;
      if constexpr (X3) {
        // the chunk's 64 tokens are summed from zero and then added, one
        // float32 rounding of the running sum per chunk
        uint4 vh[2][NCT], vl[2][NCT];
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
          for (int j = 0; j < NCT; ++j) {
            vh[s][j] = load_vt(vt, s, j);
            vl[s][j] = load_vt(vt + kVPlane, s, j);
          }
#pragma unroll
        for (int t = 0; t < GT; ++t) {
          if (t >= tiles) break;
          asm volatile("" ::: "memory");  // (operands are read where they are used)
          float gv[2][8];
          make_g(kt, 0, t, gv[0]);
          make_g(kt, 1, t, gv[1]);
#pragma unroll
          for (int i = 0; i < R; ++i) {
            f32x4 d[NCT];
#pragma unroll
            for (int j = 0; j < NCT; ++j) d[j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int s = 0; s < 2; ++s) {
              float x[8];
              load8(mr + i * kRS + 32 * s, x);
#pragma unroll
              for (int e = 0; e < 8; ++e) x[e] *= gv[s][e];
              const uint4 h = to_bf16(x), l = rest_bf16(x, h);
#pragma unroll
              for (int j = 0; j < NCT; ++j)
                d[j] = mfma_bf16(l, vh[s][j], mfma_bf16(h, vl[s][j], mfma_bf16(h, vh[s][j], d[j])));
            }
#pragma unroll
            for (int j = 0; j < NCT; ++j) acc[t][i][j] += d[j];
          }
        }
      } else {
#pragma unroll
        for (int s = 0; s < 2; ++s) {
          asm volatile("" ::: "memory");
          float gv[8], km[R][8];
          make_g(kt, s, 0, gv);
#pragma unroll
          for (int i = 0; i < R; ++i) load8(mr + i * kRS + 32 * s, km[i]);
          uint4 vb[NCT];
#pragma unroll
          for (int j = 0; j < NCT; ++j) vb[j] = load_vt(vt, s, j);
#pragma unroll
          for (int t = 0; t < GT; ++t) {
            if (t >= tiles) break;
            asm volatile("" ::: "memory");
            float gn[8];
            if (t + 1 < GT) make_g(kt, s, t + 1, gn);
#pragma unroll
            for (int i = 0; i < R; ++i) {
              float x[8];
#pragma unroll
              for (int e = 0; e < 8; ++e) x[e] = gv[e] * km[i][e];
              const uint4 h = to_bf16(x);
#pragma unroll
              for (int j = 0; j < NCT; ++j) acc[t][i][j] = mfma_bf16(h, vb[j], acc[t][i][j]);
            }
            if (t + 1 < GT)
#pragma unroll
              for (int e = 0; e < 8; ++e) gv[e] = gn[e];
          }
        }
      }
    });
    if (!live) return;
    // the sums, weighted, in the canonical layout; accumulator lane: column
    // l15, tuples 4 g4 .. +3
    const int cols = a.ones ? E : dv;
    // Table entries are fetched two tiles ahead and weights one: fetched where
    // they are used, entry, weight and store of up to 128 features ran one after
    // another, 20 us for 16 tokens (bfloat16, d = 16, P = 4).  Entries past the
    // last tile are -1.
    int4 f[2][R];
    float w[2][R][4];
    auto entries = [&](int t, int4 (&to)[R]) {
#pragma unroll
      for (int i = 0; i < R; ++i) to[i] = *(const int4*)(a.ftab + blk.tab + (t * IT + i) * 16 + 4 * g4);
    };
    auto weights = [&](const int4 (&of)[R], float (&to)[R][4]) {
#pragma unroll
      for (int i = 0; i < R; ++i) {
        const int e[4] = {of[i].x, of[i].y, of[i].z, of[i].w};
#pragma unroll
        for (int r_ = 0; r_ < 4; ++r_) to[i][r_] = a.weight[max(e[r_], 0)];
      }
    };
    entries(0, f[0]);
    if constexpr (GT > 1) entries(1, f[1]);
    weights(f[0], w[0]);
#pragma unroll
    for (int t = 0; t < GT; ++t) {
      if (t >= blk.tiles) break;
      int e[R][4];
#pragma unroll
      for (int i = 0; i < R; ++i)
        e[i][0] = f[t & 1][i].x, e[i][1] = f[t & 1][i].y, e[i][2] = f[t & 1][i].z, e[i][3] = f[t & 1][i].w;
      if (t + 1 < GT) weights(f[(t + 1) & 1], w[(t + 1) & 1]);
      if (t + 2 < GT) entries(t + 2, f[t & 1]);
#pragma unroll
      for (int i = 0; i < R; ++i)
#pragma unroll
        for (int r_ = 0; r_ < 4; ++r_) {
          if (e[i][r_] < 0) continue;
#pragma unroll
          for (int j = 0; j < NCT; ++j)
            if (16 * j + l15 < cols)
              out[(int64_t)e[i][r_] * E + 16 * j + l15] = acc[t][i][j][r_] * w[t & 1][i][r_];
        }
    }
  };
  if (wg < a.lwg) feature_block(std::integral_constant<int, IT>{});
  else feature_block(std::integral_constant<int, IT / 2>{});
}

// out[i] = sum over the parts of part[p][i], in part order.
__global__ void __launch_bounds__(256) add_parts(const float* __restrict__ part, float* __restrict__ out, int64_t count,
                                                 int parts) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= count) return;
  float s = 0.f;
  int p = 0;
  for (; p + 4 <= parts; p += 4) {  // four loads in flight
    float x[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) x[u] = part[(p + u) * count + i];
#pragma unroll
    for (int u = 0; u < 4; ++u) s += x[u];
  }
  for (; p < parts; ++p) s += part[p * count + i];
  out[i] = s;
}

template <typename T, bool X3, int NCT, int MG>
hipError_t launch_kernel(const void* k, const void* v, const StateArgs& a, int parts, hipStream_t s) {
  constexpr int PL = X3 ? 2 : 1;
  const size_t buf = (size_t)(a.dk + 1) * kRS * 4 + (size_t)PL * kCh * v_row(NCT) * 2;
  const size_t lds = 2 * buf;  // at most 76,320 bytes (d_k = d_v = 64, split operands)
  auto kern = prefill_state_kernel<T, X3, NCT, MG>;
  if (lds > 64 * 1024) {
    hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  const unsigned heads = a.by_xcd ? (a.BH + 7) / 8 * 8 : a.BH;
  hipLaunchKernelGGL(kern, dim3(heads * (unsigned)a.nwg, (unsigned)parts), dim3(kNW * 64), lds, s, (const T*)k,
                     (const T*)v, a);
  return hipGetLastError();
}

template <typename T, bool X3, int NCT>
hipError_t launch_mg(const void* k, const void* v, const StateArgs& a, int parts, hipStream_t s) {
  switch (a.mg) {
    case 1: return launch_kernel<T, X3, NCT, 1>(k, v, a, parts, s);
    case 2: return launch_kernel<T, X3, NCT, 2>(k, v, a, parts, s);
    default: return launch_kernel<T, X3, NCT, 0>(k, v, a, parts, s);
  }
}

template <typename T, bool X3>
hipError_t launch_nct(int nct, const void* k, const void* v, const StateArgs& a, int parts, hipStream_t s) {
  switch (nct) {
    case 1: return launch_mg<T, X3, 1>(k, v, a, parts, s);
    case 2: return launch_mg<T, X3, 2>(k, v, a, parts, s);
    case 3: return launch_mg<T, X3, 3>(k, v, a, parts, s);
    default: return launch_mg<T, X3, 4>(k, v, a, parts, s);
  }
}

}  // namespace

StateTable make_state_table(int dk, int P, const StateShape& shape) { return build_state_table(dk, P, shape, kNW); }

StatePlan plan_prefill_state(int64_t D, int BH, int n, int dv, bool bf16, int nwg, size_t scratch) {
  StatePlan p;
  p.nct = (dv + 15) / 16;
  p.shape = state_shape(dv, !bf16);
  p.parts = 1;
  p.part_len = std::max(kCh, (n + kCh - 1) / kCh * kCh);
  // Two workgroups fit a compute unit.  Below four rounds of them the tokens
  // are cut into parts of at least 256.
  const size_t state = sizeof(float) * (size_t)BH * D * (dv + 1);
  const int64_t wgs = (int64_t)nwg * BH;
  int parts = 1;
  while (parts < 64 && wgs * parts * 2 <= 2048 && n / (2 * parts) >= 256 && state * 2 * parts <= scratch)
    parts *= 2;
  if (parts > 1) {
    p.part_len = ((n + parts - 1) / parts + kCh - 1) / kCh * kCh;
    p.parts = (n + p.part_len - 1) / p.part_len;
    if (p.parts > 1) p.partial_bytes = state * (size_t)p.parts;
  }
  return p;
}

hipError_t launch_prefill_state(const void* k, const void* v, bool bf16, int BH, int n, int dk, int dv, int P,
                                const DevTable& t, const DevStateTable& st, const StatePlan& plan, float* S_out,
                                float* partial, hipStream_t s) {
  StateArgs a;
  a.gsym = st.gsym;
  a.list = st.list;
  a.ftab = st.ftab;
  a.ztab = st.ztab;
  a.weight = t.weight;
  a.out = plan.parts > 1 ? partial : S_out;
  a.D = t.D;
  a.BH = BH;
  a.n = n;
  a.dk = dk;
  a.dv = dv;
  a.part_len = plan.part_len;
  a.nwg = (st.blocks + st.zblocks) / kNW;
  a.lwg = st.tall / kNW;
  a.zwg = st.blocks / kNW;
  a.zcols = st.zcols;
  a.mg = P > 2 ? P - 2 : 1;
  a.by_xcd = BH >= 8;
  a.ones = !plan.shape.normalisers;
  hipError_t e = bf16 ? launch_nct<u16, false>(plan.nct, k, v, a, plan.parts, s)
                      : launch_nct<float, true>(plan.nct, k, v, a, plan.parts, s);
  if (e != hipSuccess || plan.parts == 1) return e;
  const int64_t count = (int64_t)BH * t.D * (dv + 1);
  hipLaunchKernelGGL(add_parts, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, s, partial, S_out, count,
                     plan.parts);
  return hipGetLastError();
}

}  // namespace sata
