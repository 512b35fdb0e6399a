// Host-side work list of the state sum S = sum_t phi(k_t) (x) [v_t, 1]
// (prefill_state.hip).
//
// Degree padding.  Over the d coordinates and a symbol d whose value is 1,
// every monomial of degree 0..P-1 is a sorted tuple of exactly m = P - 1
// symbols.  A feature is split as (i1, g): its smallest symbol i1 and the
// remaining (m - 1)-tuple g, all of whose symbols are >= i1.  With the tuples g
// ordered by their smallest symbol, largest first, those that go with one i1
// are a prefix of the list, so tiles of 16 consecutive g times one i1 cover
// the features with little padding.  At m = 1 the tuples g are the symbols
// themselves and the only multiplier is the symbol d.
//
// A block is `tiles` <= gt consecutive g tiles times the `rows` <= it
// multipliers from i0 on (the tiles that go with i0 are those that go with any
// of them).  ftab[tab + (t * it + i) * 16 + row] is the feature of multiplier
// i0 + i and tuple `row` of tile g0 + t (-1: none).  Blocks of more than it / 2
// rows come first, in workgroups of their own, then the others, each fullest
// first, so that the waves of a workgroup have like amounts of work.
// A normaliser block is zt g tiles (zt divides gt) whose features' normalisers
// sum_t phi_g(k_t) k_t[i1] come from one contraction with the keys:
// ztab[row of g][i1] is the feature.
#pragma once

#include <algorithm>
#include <cstdint>
#include <tuple>
#include <vector>

#include "table.hpp"

namespace sata {

// Block shape of a work list: all that the list depends on besides (d, P), so
// (d, P, shape) names a list, and the shape that a kernel assumes.
struct StateShape {
  int gt = 0, it = 0;        // g tiles and multipliers of a feature block
  int zt = 0;                // g tiles of a normaliser block
  bool normalisers = false;  // normalisers from blocks of their own
  bool operator<(const StateShape& o) const {
    return std::tie(gt, it, zt, normalisers) < std::tie(o.gt, o.it, o.zt, o.normalisers);
  }
};

// Feature blocks: gt * it * (column tiles) accumulator tiles (4 registers each)
// beside the operands at two waves per SIMD; normaliser blocks: up to 5
// accumulator tiles per g tile.  split: split operands (float32 inputs).
constexpr int state_gt(int col_tiles, bool split) { return split ? (col_tiles <= 2 ? 4 : 2) : (col_tiles == 1 ? 8 : 4); }
constexpr int state_it(int col_tiles, bool split) { return split ? (col_tiles == 1 ? 4 : 2) : (col_tiles <= 2 ? 4 : 2); }
constexpr int state_zt(bool split) { return split ? 2 : 4; }

// The shape for values of d_v columns.
inline StateShape state_shape(int dv, bool split) {
  const int nct = (dv + 15) / 16;
  StateShape s;
  s.gt = state_gt(nct, split);
  s.it = state_it(nct, split);
  s.zt = state_zt(split);
  s.normalisers = dv % 16 == 0;
  return s;
}

struct StateBlock {
  int32_t g0, i0;
  int32_t rows, tiles;
  int32_t tab;
};

struct StateTable {
  int gtiles = 0;                  // tiles of 16 tuples g, padded to whole blocks
  int zcols = 0;                   // multipliers d + 1 rounded up to 16
  int tall = 0, blocks = 0, zblocks = 0;  // padded to whole workgroups; blocks counts the tall ones too
  std::vector<uint64_t> gsym;      // [gtiles * 16] symbols of g, one a byte (unused: d)
  std::vector<StateBlock> list;    // the blocks, then the normaliser blocks
  std::vector<int32_t> ftab;
  std::vector<int32_t> ztab;       // [gtiles * 16][zcols]
};

// Position of the sorted tuple t[0..m) over symbols 0..d (the trailing ones
// equal to d left out) in the library's feature order.
inline int64_t feature_rank(int d, const int* t, int m) {
  int p = m;
  while (p > 0 && t[p - 1] == d) --p;
  int64_t r = 0;
  for (int e = 0; e < p; ++e) r += binom((int64_t)d + e - 1, e);  // lower degrees
  int lo = 0;
  for (int j = 0; j < p; ++j) {
    // tuples that agree before j and have a smaller symbol x at j: the rest
    // runs over x..d-1
    for (int x = lo; x < t[j]; ++x) r += binom((int64_t)(d - x) + (p - j - 1) - 1, p - j - 1);
    lo = t[j];
  }
  return r;
}

// cum[r][x]: non-decreasing r-tuples over symbols y..d-1, summed over y < x (the
// steps of feature_rank).
struct RankSums {
  std::vector<int64_t> cum[kMaxP];
  int64_t base[kMaxP + 1] = {0};  // features of lower degrees
  explicit RankSums(int d) {
    for (int r = 0; r < kMaxP; ++r) {
      cum[r].assign((size_t)d + 1, 0);
      for (int x = 0; x < d; ++x) cum[r][(size_t)x + 1] = cum[r][(size_t)x] + binom((int64_t)(d - x) + r - 1, r);
      base[r + 1] = base[r] + binom((int64_t)d + r - 1, r);
    }
  }
};

// The list takes a few ns a feature to build: the rank of (i1, g) is a term of g
// and two of i1 (symbol by symbol and binomial by binomial it took 0.5 s for the
// 814,385 features of d = 64, P = 5, now 0.02; the feature table takes 0.04).
inline StateTable build_state_table(int d, int P, int gt, int it, int zt, bool normalisers, int waves) {
  StateTable st;
  const int m = P - 1, mg = m > 1 ? m - 1 : 1;
  // the tuples g, one symbol a byte (unused bytes: d): by their smallest symbol,
  // largest first, then in lexicographic order
  std::vector<uint64_t> gs;
  {
    std::vector<uint64_t> lex;
    std::vector<size_t> first((size_t)d + 2, 0);  // where the tuples of a smallest symbol start
    lex.reserve((size_t)binom((int64_t)d + mg, mg));
    for_each_tuple(d + 1, mg, [&](const int* t) {
      uint64_t w = 0;
      for (int j = 0; j < 8; ++j) w |= (uint64_t)(uint8_t)(j < mg ? t[j] : d) << (8 * j);
      lex.push_back(w);
      first[(size_t)t[0] + 1] = lex.size();
    });
    gs.reserve(lex.size());
    for (int s = d; s >= 0; --s) gs.insert(gs.end(), lex.begin() + first[(size_t)s], lex.begin() + first[(size_t)s + 1]);
  }
  const int ng = (int)gs.size();
  auto symbol = [&](int g, int j) { return (int)(gs[(size_t)g] >> (8 * j) & 0xff); };
  st.gtiles = ((ng + 15) / 16 + gt - 1) / gt * gt;  // whole blocks: kernels read them unchecked
  st.zcols = (d + 1 + 15) / 16 * 16;
  uint64_t none = 0;
  for (int j = 0; j < 8; ++j) none |= (uint64_t)(uint8_t)d << (8 * j);
  st.gsym = gs;
  st.gsym.resize((size_t)st.gtiles * 16, none);
  // the part of a feature's rank that is the tuple's, and the tuple's degree
  const RankSums rs(d);
  std::vector<int64_t> rank((size_t)ng);
  std::vector<uint8_t> degree((size_t)ng);
  for (int g = 0; g < ng; ++g) {
    int p = mg;
    while (p > 0 && symbol(g, p - 1) == d) --p;
    int64_t r = rs.base[p + 1];
    for (int j = 0; j < p; ++j) {
      const std::vector<int64_t>& c = rs.cum[p - j - 1];
      r += c[(size_t)symbol(g, j)] - (j ? c[(size_t)symbol(g, j - 1)] : 0);
    }
    rank[(size_t)g] = r;
    degree[(size_t)g] = (uint8_t)p;
  }
  auto feature = [&](int g, int i1) -> int32_t {
    if (g >= ng) return -1;
    const int g0 = symbol(g, 0), p = degree[(size_t)g];
    if (m == 1) return i1 == d ? (g0 == d ? 0 : 1 + g0) : -1;  // the tuples g are the features
    if (i1 > g0) return -1;
    if (i1 == d) return 0;
    return (int32_t)(rank[(size_t)g] + rs.cum[p][(size_t)i1] - (p > 0 ? rs.cum[p - 1][(size_t)i1] : 0));
  };
  std::vector<StateBlock> low;
  for (int g0 = 0; g0 < st.gtiles; g0 += gt) {
    const int top = m == 1 ? d : symbol(g0 * 16, 0);  // the largest multiplier of these tiles
    for (int i0 = m == 1 ? d : 0; i0 <= top; i0 += it) {
      StateBlock b{g0, i0, std::min(it, top + 1 - i0), 0, (int32_t)st.ftab.size()};
      st.ftab.resize(st.ftab.size() + (size_t)gt * it * 16, -1);
      int32_t* f = st.ftab.data() + b.tab;
      for (int t = 0; t < gt; ++t)
        for (int i = 0; i < it; ++i)
          for (int r = 0; r < 16; ++r, ++f) {
            if (i0 + i <= top) *f = feature((g0 + t) * 16 + r, i0 + i);
            if (*f >= 0) b.tiles = t + 1;
          }
      (2 * b.rows > it ? st.list : low).push_back(b);
    }
  }
  auto order = [&](std::vector<StateBlock>& v) {
    std::stable_sort(v.begin(), v.end(), [](const StateBlock& x, const StateBlock& y) { return x.tiles > y.tiles; });
    while (v.size() % (size_t)waves) v.push_back({-1, 0, 0, 0, 0});
  };
  order(st.list);
  st.tall = (int)st.list.size();
  order(low);
  st.list.insert(st.list.end(), low.begin(), low.end());
  st.blocks = (int)st.list.size();
  if (normalisers) {
    for (int g0 = 0; g0 < st.gtiles; g0 += zt) st.list.push_back({g0, 0, 0, zt, 0});
    while (st.list.size() % (size_t)waves) st.list.push_back({-1, 0, 0, 0, 0});
    st.ztab.resize((size_t)st.gtiles * 16 * st.zcols);
    for (int g = 0; g < st.gtiles * 16; ++g)
      for (int i = 0; i < st.zcols; ++i)
        st.ztab[(size_t)g * st.zcols + i] = i <= d ? feature(g, i) : -1;
  }
  st.zblocks = (int)st.list.size() - st.blocks;
  return st;
}

inline StateTable build_state_table(int d, int P, const StateShape& s, int waves) {
  return build_state_table(d, P, s.gt, s.it, s.zt, s.normalisers, waves);
}

}  // namespace sata
