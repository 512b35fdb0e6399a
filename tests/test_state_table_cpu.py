"""The work list of the state sum (state_table.hpp), built by its own host code:
every feature is held by exactly one (block, multiplier, tuple) slot and by
exactly one normaliser slot, the slot's symbols are the feature's indices, and
blocks are dealt to workgroups as the kernel assumes."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2602_00294_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include <set>
#include "state_table.hpp"
using namespace sata;
int main() {
  int bad = 0;
  for (int d : {1, 2, 3, 8, 16, 17, 24, 33, 64})
    for (int P = 2; P <= 8; ++P) {
      const int64_t D = feature_count(d, P);
      if (D > 50000) continue;
      const FeatureTable F = build_table(d, P);
      for (int64_t f = 0; f < D; f += 1 + D / 97) {  // feature_rank against the table's order
        int t[kMaxP];
        const int p = packed_degree(F.packed[f]);
        for (int j = 0; j < P - 1; ++j) t[j] = j < p ? packed_index(F.packed[f], j) : d;
        bad += feature_rank(d, t, P - 1) != f;
      }
      for (int gt : {2, 4, 8})
        for (int it : {2, 4})
          for (int zt : {2, 4}) {
            if (zt > gt) continue;
            const StateTable t = build_state_table(d, P, gt, it, zt, true, 4);
            std::vector<int> seen(D, 0), zseen(D, 0);
            bad += t.tall % 4 || t.blocks % 4 || t.zblocks % 4 || (int)t.list.size() != t.blocks + t.zblocks;
            bad += t.gtiles % gt || (int)t.gsym.size() != 16 * t.gtiles;
            auto symbols = [&](int g, int i1) {
              std::multiset<int> s;
              for (int j = 0; j < (P > 2 ? P - 2 : 1); ++j) s.insert((int)(t.gsym[g] >> (8 * j) & 255));
              s.insert(i1);
              s.erase(d);
              return s;
            };
            auto indices = [&](int f) {
              std::multiset<int> s;
              for (int j = 0; j < packed_degree(F.packed[f]); ++j) s.insert(packed_index(F.packed[f], j));
              return s;
            };
            for (int b = 0; b < t.blocks; ++b) {
              const StateBlock& B = t.list[b];
              if (B.g0 < 0) continue;
              bad += B.g0 + gt > t.gtiles || B.i0 + B.rows > d + 1 || (b < t.tall) != (2 * B.rows > it);
              for (int x = 0; x < gt; ++x)
                for (int i = 0; i < it; ++i)
                  for (int r = 0; r < 16; ++r) {
                    const int f = t.ftab[B.tab + (x * it + i) * 16 + r];
                    if (f < 0) continue;
                    ++seen[f];
                    bad += x >= B.tiles || i >= B.rows || symbols((B.g0 + x) * 16 + r, B.i0 + i) != indices(f);
                  }
            }
            std::set<int> tiles;
            for (int b = t.blocks; b < (int)t.list.size(); ++b)
              if (t.list[b].g0 >= 0)
                for (int x = 0; x < zt; ++x) bad += !tiles.insert(t.list[b].g0 + x).second;
            bad += (int)tiles.size() != t.gtiles || *tiles.rbegin() != t.gtiles - 1;
            for (int g = 0; g < 16 * t.gtiles; ++g)
              for (int i = 0; i < t.zcols; ++i) {
                const int f = t.ztab[(size_t)g * t.zcols + i];
                if (f < 0) continue;
                ++zseen[f];
                bad += i > d || symbols(g, i) != indices(f);
              }
            for (int64_t f = 0; f < D; ++f) bad += seen[f] != 1 || zseen[f] != 1;
          }
    }
  std::printf("%d\n", bad);
  return bad != 0;
}
"""

# Every call's list comes out of one cache keyed by (d, P, shape), filled in
# either order of bfloat16 and float32 and of d_v: it has to be the list that
# the call's kernel walks, with its number of g tiles per normaliser block.
CACHE_PROGRAM = r"""
#include <cstdio>
#include <map>
#include "state_table.hpp"
using namespace sata;
int main() {
  int bad = 0;
  for (int d : {8, 32})
    for (int order = 0; order < 2; ++order) {
      const int P = 4;
      const int64_t D = feature_count(d, P);
      std::map<std::tuple<int, int, StateShape>, StateTable> cache;
      for (int i = 0; i < 128; ++i) {
        const int call = order ? 127 - i : i, dv = call / 2 + 1;
        const bool split = call % 2;
        const StateShape s = state_shape(dv, split);
        bad += s.zt != state_zt(split) || s.gt != state_gt((dv + 15) / 16, split) ||
               s.it != state_it((dv + 15) / 16, split) || s.normalisers != (dv % 16 == 0);
        const auto key = std::make_tuple(d, P, s);
        auto it = cache.find(key);
        if (it == cache.end()) it = cache.emplace(key, build_state_table(d, P, s, 4)).first;
        const StateTable& t = it->second;
        std::vector<int> seen(D, 0);
        for (int b = t.blocks; b < (int)t.list.size(); ++b) {
          const StateBlock& B = t.list[b];
          if (B.g0 < 0) continue;
          bad += B.g0 + state_zt(split) > t.gtiles;
          for (int x = 0; x < state_zt(split) && B.g0 + x < t.gtiles; ++x)
            for (int r = 0; r < 16; ++r)
              for (int z = 0; z < t.zcols; ++z) {
                const int f = t.ztab[(size_t)((B.g0 + x) * 16 + r) * t.zcols + z];
                if (f >= 0) ++seen[f];
              }
        }
        for (int64_t f = 0; f < D; ++f) bad += seen[f] != (dv % 16 == 0);
      }
    }
  std::printf("%d\n", bad);
  return bad != 0;
}
"""

# A first call at new sizes waits for its tables: the work list has to be no
# longer in the making than a few times the feature table of the same sizes.
TIME_PROGRAM = r"""
#include <chrono>
#include <cstdio>
#include "state_table.hpp"
using namespace sata;
template <typename F> double best(F&& f) {
  double b = 1e9;
  for (int i = 0; i < 3; ++i) {
    const auto t0 = std::chrono::steady_clock::now();
    f();
    b = std::min(b, std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count());
  }
  return b;
}
int main() {
  int bad = 0;
  size_t used = 0;
  for (int i = 0; i < 2; ++i) {
    const int d = i ? 20 : 64, P = i ? 8 : 5;
    const double features = best([&] { used += build_gen_program(build_table(d, P), 4096, 32).size(); });
    const double list = best([&] { used += build_state_table(d, P, state_shape(16, i), 4).ftab.size(); });
    std::printf("d=%d P=%d: feature table %.4f s, work list %.4f s\n", d, P, features, list);
    bad += list > 4 * features;
  }
  return bad != 0 || used == 0;
}
"""


def _run(tmp_path, program):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no g++")
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(program)
    subprocess.run([gxx, "-O1", "-std=c++17", f"-I{CSRC}", str(src), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout


def test_state_table_holds_every_feature_once(tmp_path):
    _run(tmp_path, PROGRAM)


def test_cached_state_table_is_the_calls_own(tmp_path):
    _run(tmp_path, CACHE_PROGRAM)


def test_state_table_is_quick_to_build(tmp_path):
    _run(tmp_path, TIME_PROGRAM)
