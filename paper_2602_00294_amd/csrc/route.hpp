// Host-side estimates, in microseconds on an MI355X, of the two ways to a
// prefill, and the choice between them.
//
// Pair by pair (prefill_direct_kernel.hpp, then prefill_state.hip where the
// state is asked for) the work grows with n^2; a workgroup walks all chunks of
// 64 keys up to its queries.  The chunked scan's work grows with n D; a
// workgroup walks all chunks of its part of the sequence for its slice of the
// features.  So each side takes the longer of two times: that of all its work
// on the whole chip, and that of one workgroup's chain of chunks, which is what
// short calls and calls with few heads wait for.
//
// The constants were fitted to 5230 calls timed both ways (d = 8 .. 64, P = 2 ..
// 8, 1 .. 1024 heads, 16 .. 65536 tokens, d_k != d_v and rows without vectors
// among them), with and without the state: the estimates are within 14% for two
// calls of three; the pairs were taken and slower by more than 4% in 26 of the
// 10460 (by at most 17%), the scan by more than 20% in 91.  Before, with a share
// of D for the scan and no chains, the pairs were slower by more than 5% in 647
// of 2340 other calls with a state, now in 20.  Some, us pair by pair / scan:
//   d  P  dtype heads     n   with the state    y alone
//   16 4  bf16    8      64       18 /   28      13 /  21
//   16 4  bf16   64    2048      115 /  307      48 / 302
//   32 2  bf16    1   65536      774 /  426     736 / 427
//    8 3  f32     8   16384      343 /  146     339 / 145
//   32 4  f32     8    4096      218 /  508      98 / 498
//   32 2  f32   256    1024      299 /  167     245 / 166
//   64 3  f32     1   16384      674 /  295     605 / 294
#pragma once

#include <algorithm>
#include <cstdint>

#include "state_table.hpp"
#include "table.hpp"

namespace sata {

// Query tiles per wave of the pair-by-pair kernel: many reuse a chunk's
// operands; one where larger blocks would leave compute units without work.
constexpr int direct_wide_tiles(bool split, int col_tiles) { return split || col_tiles >= 4 ? 2 : 3; }
inline int direct_query_tiles(bool split, int dv, int heads, int n) {
  const int wide = direct_wide_tiles(split, (dv + 16) / 16);
  return ((int64_t)n + 64 * wide - 1) / (64 * wide) * heads >= 512 ? wide : 1;
}

// A grid of the pairs' kernels: heads in eights (one per XCD) times blocks of
// rows.  HIP launches fewer than 2^32 threads, of which a block has 256.
constexpr int64_t kMaxPairBlocks = ((int64_t)1 << 24) - 1;
inline int64_t pair_blocks(int heads, int n, int rows_per_block) {
  return ((int64_t)n + rows_per_block - 1) / rows_per_block * (heads >= 8 ? ((int64_t)heads + 7) / 8 * 8 : heads);
}
inline int64_t direct_blocks(bool split, int dv, int query_heads, int n) {
  return pair_blocks(query_heads, n, 64 * direct_query_tiles(split, dv, query_heads, n));
}
// Own rows' tiles per wave of the pair-by-pair backward: two share the staged
// rows' operands; one where that would leave compute units without work, or
// (float32) registers short.
inline int backward_tiles(bool bf16, int heads, int n) {
  return bf16 && ((int64_t)n + 127) / 128 * heads >= 512 ? 2 : 1;
}
inline int64_t backward_blocks(bool bf16, int heads, int n) {
  return pair_blocks(heads, n, 64 * backward_tiles(bf16, heads, n));
}

struct RouteCall {
  bool bf16 = false;
  int dk = 0, dv = 0, P = 0;
  int64_t D = 0;
  int heads = 0;        // key/value heads
  int n = 0;            // tokens
  bool vectors = true;  // rows of q, k and v are whole aligned 16-byte vectors
};

// What of the scan's plan its time depends on.
struct ScanShape {
  bool tuned = false;     // one of the kernels for P = 4, d in {16, 32}; else generated features:
  int chunk = 64;         // (tuned) tokens per chunk
  int wave_features = 0;  // features of the busiest wave
  int slices = 1;         // workgroups per head and part
  int parts = 1;          // parts of the sequence side by side
};

// Work on the whole chip and one chain of it overlap all but fully.
inline double longer_of(double a, double b) { return std::max(a, b) + 0.25 * std::min(a, b); }

// The outputs, pair by pair: c ps a pair and `own` ps a token (the query's own
// chunk) on the whole chip; tau us a chunk in a chain.  Rows that are no whole
// vectors are staged element by element.
inline double pairs_us(const RouteCall& r) {
  const int nct = (r.dv + 16) / 16, terms = std::max(0, r.P - 4);
  double c, own, tau, start;
  if (r.bf16) {
    c = 0.08 + 0.03 * nct + (r.dk > 32 ? 0.06 : 0.0) + 0.06 * terms;
    own = 10.0 + 20.0 * nct;
    tau = 0.42 + 0.06 * nct + 0.09 * terms;
    start = 6.5;
    if (!r.vectors) c *= 4.5, own *= 2.0, tau *= 5.0;
  } else {
    if (r.dk <= 16) {
      c = 0.19 + 0.10 * nct + 0.05 * terms;
      own = 60.0 + 85.0 * nct;
      tau = 0.60 + 0.18 * nct;
      start = 8.0 + 1.4 * nct;
    } else if (r.dk <= 32) {
      c = 0.26 + 0.14 * nct + 0.1 * terms;
      own = 220.0 + 70.0 * nct;
      tau = 0.97 + 0.09 * nct;
      start = 10.5 + 1.2 * nct;
    } else {
      c = 0.33 + 0.23 * nct + 0.1 * terms;
      own = 200.0 + 235.0 * nct;
      tau = 1.10 + 0.23 * nct;
      start = 15.5 + 1.4 * nct;
    }
    tau += 0.11 * terms;
    if (!r.vectors) c *= 1.9, own *= 1.3, tau *= 2.5;
  }
  const int tiles = direct_query_tiles(!r.bf16, r.dv, r.heads, r.n);
  const double chunks = (r.n + 63) / 64, tokens = (double)r.heads * r.n;
  const double t = start + longer_of(tokens * (c * 0.5 * r.n + own) * 1e-6,
                                     chunks * tau * (1.0 + (r.bf16 ? 0.25 : 0.4) * (tiles - 1)));
  return std::max(13.8, r.bf16 ? t : 1.04 * t);  // (13.8: calls one after another)
}

// Workgroups per head of the state sum, near enough without its work list.
inline double state_workgroups(const RouteCall& r) {
  const StateShape s = state_shape(r.dv, !r.bf16);
  const int mg = std::max(1, r.P - 2);
  const double gtiles = (double)((binom((int64_t)r.dk + mg, mg) + 15) / 16);
  double blocks = (double)r.D / (16 * s.gt * s.it) + 0.5 * gtiles / s.gt;
  if (r.P > 2) blocks = std::max(blocks, (r.dk + 1.0) / s.it);
  return blocks / 4 + (r.P == 2 ? 1.0 : 1.5) + (s.normalisers ? std::max(1.0, gtiles / (4 * s.zt)) : 0.0);
}

// The state as one sum, its tokens in `parts` parts: tau us a chunk and end_us at
// a block's end, both by the tiles x multipliers of a wave's block.
inline double state_us(const RouteCall& r, double workgroups, int parts) {
  const StateShape s = state_shape(r.dv, !r.bf16);
  const int mg = std::max(1, r.P - 2), at = std::min((r.dv + 15) / 16, 3) - 1;
  const double gtiles = (double)((binom((int64_t)r.dk + mg, mg) + 15) / 16);
  const double slots = std::min<double>(s.gt, gtiles) * (r.P == 2 ? 1 : std::min(s.it, r.dk + 1));
  static constexpr double kTau[2][3] = {{0.30, 0.38, 0.62}, {0.10, 0.155, 0.29}};
  static constexpr double kEnd[2][3] = {{0.33, 1.0, 2.0}, {0.18, 0.55, 1.1}};   // on the whole chip
  static constexpr double kFirst[2][3] = {{0.1, 0.6, 1.8}, {0.0, 0.0, 0.0}};    // of one block
  static constexpr double kFull[2][3] = {{0.75, 1.05, 1.25}, {0.65, 0.85, 0.75}};
  double tau = (r.bf16 ? 0.1 : 0.5) + slots * kTau[r.bf16][at];
  if (r.P > 4) tau *= r.bf16 ? 1.5 + 0.2 * (r.P - 5) : 1.15 + 0.1 * (r.P - 5);
  if (!r.vectors) tau *= 1.8;
  const double chunks = (r.n + 64 * parts - 1) / (64 * parts);
  const double rounds = workgroups * r.heads * parts / 512.0;
  double t = 2.0 + longer_of(slots * kFirst[r.bf16][at] + chunks * tau,
                             rounds * (slots * kEnd[r.bf16][at] + chunks * tau * kFull[r.bf16][at]));
  if (parts > 1) t += (r.bf16 ? 7.0 : 2.0) + 1.6e-6 * parts * r.heads * (double)r.D * (r.dv + 1);
  return t;
}

// The chunked scan, outputs and state.
inline double scan_us(const RouteCall& r, const ScanShape& s) {
  const double chunks = (r.n + 63) / 64, state_bytes = 4.0 * r.heads * (double)r.D * (r.dv + 1);
  if (s.tuned) {
    // per 64 tokens: one head, and 256 heads
    double chain, chip;
    if (r.dk > 16) {
      chain = s.chunk == 64 ? 8.2 : s.chunk == 32 ? 19.3 : 15.2;
      chip = s.chunk == 64 ? 34.0 : s.chunk == 32 ? 84.0 : 76.0;
      return 50.0 + chunks * std::max(chain, chip * r.heads / 256.0) + 5e-7 * state_bytes;
    }
    chain = s.chunk == 64 ? 8.4 : s.chunk == 32 ? 11.3 : 9.2;
    chip = s.chunk == 64 ? 8.1 : s.chunk == 32 ? 10.0 : 12.6;
    return (s.chunk == 128 ? 28.0 : 18.0) + chunks * std::max(chain, chip * r.heads / 256.0) + 3e-7 * state_bytes;
  }
  const int nct = (r.dv + 16) / 16;
  double feature = r.bf16 ? 0.045 + 0.028 * nct : 0.09 + 0.035 * nct;
  if (r.P > 4) feature += r.bf16 ? 0.04 + 0.035 * (r.P - 4) : 0.05 + 0.045 * (r.P - 4);
  double chunk = std::max(r.bf16 ? 3.2 : 4.7, 0.8 + s.wave_features * feature);
  if (!r.vectors) chunk *= 1.2;
  // rounds of one workgroup per compute unit; in parts, a first pass sums them
  double rounds = (double)s.slices * r.heads * s.parts / 256.0;
  rounds = std::max(1.0, rounds <= 4.0 ? (double)(int64_t)(rounds + 0.9999) : rounds);
  const double passes = s.parts == 1 ? 1.0 : r.bf16 ? 1.55 : 1.45;
  const double start = 12.0 + (s.slices > 1 ? 4.0 : 0.0) + (s.wave_features > 32 ? 8.0 : 0.0) + 1e-7 * state_bytes;
  const double part_chunks = (r.n + 64 * s.parts - 1) / (64 * s.parts);
  return std::max(17.5, start + passes * part_chunks * chunk * rounds + 5e-6 * r.heads * (double)r.n * r.dv);
}

}  // namespace sata
