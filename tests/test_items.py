"""Which item a workgroup takes: division by multiplication, and the items of a launch each taken exactly once; classes of
tiles and live rows from bounds that a wave works out once."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(__file__), "..", "paper_2410_01485_amd", "csrc")
PROGRAM = r"""
#include <cstdio>
#include <vector>
#include "lg_mask.h"
int main() {
  const int ds[] = {1, 2, 3, 5, 7, 8, 12, 63, 64, 65, 1000, 4097, 65535, 65536, 16777215, 715827883, 1073741824, 2147483646, 2147483647};
  for (int d : ds) {
    const LgDiv v = lg_make_div(d);
    std::vector<long long> ns = {0, 1, 2147483646, 2147483647};
    for (long long q = 1; q * d - 1 <= 2147483647LL && q < 4000; q = q < 50 ? q + 1 : q * 3 / 2)
      for (int e = -1; e <= 1; ++e) ns.push_back(q * d + e);
    for (long long q = 2147483647LL / d, k = 0; k < 50 && q - k > 0; ++k)
      for (int e = -1; e <= 1; ++e) ns.push_back((q - k) * d + e);
    for (long long n : ns) {
      if (n < 0 || n > 2147483647LL) continue;
      int rem, x = lg_divmod(v, (int)n, &rem);
      if (x != n / d || rem != n % d) { std::printf("%lld / %d = %d rest %d\n", n, d, x, rem); return 1; }
    }
  }
  const int shapes[][5] = {{1, 1, 1, 1, 1}, {2, 8, 2, 5, 3}, {3, 6, 6, 7, 16}, {1, 64, 8, 129, 1000}, {4, 4, 1, 2, 2}, {4, 16, 16, 8, 7}, {4, 32, 16, 2, 300}, {1, 32, 32, 5, 20}, {3, 64, 32, 6, 144}, {2, 32, 32, 1, 8}, {4, 24, 24, 64, 768}, {1, 32, 32, 65, 260}, {100, 32, 32, 2, 800}, {31, 64, 64, 3, 700}, {20, 32, 32, 6, 333}};
  for (auto& s : shapes) {
    const int B = s[0], Hq = s[1], Hkv = s[2], nqt = s[3], run = s[4], total = B * Hq * nqt;
    const LgItems w = lg_make_items(total, run, nqt, Hq, Hkv, B % 2 ? 64 : 128);
    std::vector<int> seen(total, 0);
    for (long long id = 0; id < lg_run_grid(total, run); ++id) {
      const int L = lg_item_of((int)id, w.run);
      if (L >= total) continue;
      const LgItem it = lg_item(w, L);
      if (it.b < 0 || it.b >= B || it.hq < 0 || it.hq >= Hq || it.x < 0 || it.x >= nqt || it.hk != it.hq / (Hq / Hkv)) return 2;
      ++seen[(it.b * Hq + it.hq) * nqt + it.x];
    }
    for (int x : seen)
      if (x != 1) return 3;
  }
  return 0;
}
"""

RUNS = r"""
#include <cstdio>
#include <vector>
#include "lg_mask.h"
// B, Hq, Hkv, N, sink, window, block, stride: causal, windowed and strided, few heads and many, one tile and hundreds
int main() {
  const int shapes[][8] = {{1, 8, 2, 12000, 0, 12000, 1, 0}, {1, 12, 4, 16000, 0, 16000, 1, 0}, {1, 16, 4, 5000, 64, 2600, 1, 0},
                           {2, 4, 1, 12000, 0, 12000, 1, 0}, {3, 2, 2, 30000, 0, 30000, 1, 0}, {1, 4, 2, 9000, 64, 512, 64, 8}, {1, 1, 1, 9000, 0, 9000, 1, 0},
                           {1, 1, 1, 70, 0, 70, 1, 0}, {100, 3, 1, 300, 0, 300, 1, 0}, {1, 6, 6, 2200, 0, 2200, 1, 0}, {5, 3, 3, 128, 0, 128, 1, 0},
                           {1, 7, 1, 4000, 0, 600, 1, 0}, {2, 16, 4, 3000, 16, 3000, 1, 0}, {4, 8, 4, 1000, 0, 1000, 1, 0}, {1, 64, 4, 33000, 64, 9000, 1, 0}};
  for (auto& s : shapes) {
    const int B = s[0], Hq = s[1], Hkv = s[2], N = s[3], G = Hq / Hkv, tiles = (N + 127) / 128, total = tiles * Hq * B;
    const LgMask m = lg_make_mask(N, s[4], s[5], s[6], s[7]);
    for (int varied = 0; varied < 2; ++varied) {
      const LgRuns w = lg_runs(m, B * Hkv, tiles, G, varied);
      const LgItems items = lg_make_items(total, w, tiles, Hq, Hkv, 128);
      const long long grid = lg_run_grid(w, total);
      std::vector<int> seen(total, 0);
      double work[8] = {}, all = 0, longest = 0;
      for (long long id = 0; id < grid; ++id) {
        const int L = lg_item_of((int)id, w);
        if (L != lg_item_of((int)id, items)) return 1;
        if (L < 0 || L >= total) continue;
        ++seen[L];
        const LgItem it = lg_item(items, L);
        const int qt = tiles - 1 - it.x, q0 = qt * 128, q1 = q0 + 127 < N - 1 ? q0 + 127 : N - 1;
        const LgQSched qs = lg_qsched_init(m, q0, q1);
        double keys = 4;  // (start and end of an item, in tiles)
        for (int t = lg_qsched_next(m, qs, -1); t >= 0; t = lg_qsched_next(m, qs, t)) ++keys;
        work[id & 7] += keys;
        all += keys;
        longest = keys > longest ? keys : longest;
      }
      for (int x : seen)
        if (x != 1) return 2;
      // workgroups without an item: less than an eighth, beyond the padding to whole rounds of runs
      if (grid > total + total / 8 + 8LL * w.run) { std::printf("grid %lld for %d items\n", grid, total); return 3; }
      // no XCD has much more than its share (a launch that each XCD gets a few rows of: not more than those; one with a CU for
      // every workgroup: no matter)
      double most = 0;
      for (double x : work) most = x > most ? x : most;
      if (!varied && total > 256 && most > 1.3 * all / 8 && most > 8 * longest) {
        std::printf("B %d Hq %d Hkv %d N %d: an XCD has %.0f of %.0f tiles\n", B, Hq, Hkv, N, most, all / 8);
        return 4;
      }
    }
  }
  return 0;
}
"""

ORDER = r"""
#include <cstdio>
#include <vector>
#include "lg_mask.h"
// Causal heads, every XCD an eighth of them: the shares of its four shader engines, which get workgroups in turn, and, where
// all are in flight at once, of its 32 CUs.
int main() {
  const int heads_[] = {32, 64, 128, 512, 2048}, tiles_[] = {3, 4, 8, 16, 24, 28, 36, 47, 64};
  for (int heads : heads_)
    for (int tiles : tiles_) {
      const int total = heads * tiles, each = total / 8;
      const LgItems w = lg_make_items(total, each, tiles, heads, heads, heads == 64 ? 64 : 128);
      double se[4] = {}, cu[32] = {}, all = 0;
      std::vector<int> seen(total, 0);
      int changes = 0, before = 0;
      for (int i = 0; i < each; ++i) {
        const LgItem it = lg_item(w, lg_item_of(8 * i, w));  // XCD 0
        changes += it.hk != before;
        before = it.hk;
        if (it.hk >= heads / 8) return 1;                    // whole heads
        const double cost = tiles - it.x + 1;
        ++seen[it.hk * tiles + it.x];
        se[i % 4] += cost;
        cu[i % 32] += cost;
        all += cost;
      }
      for (int x = 0; x < each; ++x)
        if (seen[x] != 1) return 2;
      // in launches of many rounds, whose keys would outgrow an L2 otherwise, one head after the other
      if (total > 4096 && changes != heads / 8 - 1) return 5;
      for (double x : se)
        if (x > 1.08 * all / 4) { std::printf("%d heads of %d tiles: an engine has %.0f of %.0f\n", heads, tiles, x, all / 4); return 3; }
      if (each == 96 || each == 128)
        for (double x : cu)
          if (x > 1.3 * all / 32) { std::printf("%d heads of %d tiles: a CU has %.0f of %.1f\n", heads, tiles, x, all / 32); return 4; }
    }
  return 0;
}
"""

KINDS = r"""
#include <cstdio>
#include <cstdlib>
#include "lg_mask.h"
// classes and runs from bounds worked out once, against the general class and the predicate
int main() {
  std::srand(5);
  auto rnd = [](int n) { return std::rand() % n; };
  const int blocks[] = {1, 1, 2, 16, 48, 64, 100}, strides[] = {0, 0, 0, 1, 2, 3, 8}, lens[] = {16, 32, 64};
  for (int it = 0; it < 400000; ++it) {
    const int N = 1 + rnd(it % 3 ? 300 : 3000), b = blocks[rnd(7)], st = strides[rnd(7)];
    const LgMask m = lg_make_mask(N, b * rnd(6), b * (1 + rnd(20)), b, st);
    const int q0 = rnd(N), q1 = q0 + lens[rnd(3)] - 1 < N ? q0 + lens[rnd(3)] - 1 : N - 1, qe = q1 < q0 ? q0 : (q1 < N ? q1 : N - 1);
    const int k0 = rnd(N), k1 = k0 + lens[rnd(3)] - 1;
    const int want = lg_tile_kind(m, q0, qe, k0, k1);
    if (lg_rows_kind(m, lg_rows(m, q0, qe), k0, k1) != want) { std::printf("rows: N %d b %d st %d q %d..%d k %d..%d\n", N, b, st, q0, qe, k0, k1); return 1; }
    const LgKeys ks = lg_keys(m, k0, k1);
    const int got = lg_keys_kind(ks, q0, qe);
    // (PARTIAL is allowed for FULL where some of the keys are columns; nothing else)
    if (got != want && !(got == LG_TILE_PARTIAL && want == LG_TILE_FULL && lg_has_column_key(m, k0, k1 < N ? k1 : N - 1))) {
      std::printf("keys: N %d b %d st %d q %d..%d k %d..%d got %d want %d\n", N, b, st, q0, qe, k0, k1, got, want);
      return 2;
    }
    if (lg_keys_kind(ks, N - 1 - rnd(N), N) == LG_TILE_FULL) return 3;  // rows past the end
    if (lg_keys_kind(lg_keys(m, N + rnd(50), N + 100), q0, qe) != LG_TILE_DEAD) return 4;  // keys past the end
    const int j = rnd(N), i = rnd(N);
    const bool column = j < m.sink || (m.stride > 0 && lg_strided(m, lg_div_b(m, j)));
    const unsigned seen = (unsigned)((column ? m.N : lg_window_end(m, j)) - j);
    if (((unsigned)(i - j) < seen) != lg_live(m, i, j)) { std::printf("seen: N %d b %d st %d i %d j %d\n", N, b, st, i, j); return 5; }
    const int w = (lg_div_b(m, i) - m.wb + 1) * m.b;
    const bool live = j <= i && (j >= w || j < m.sink || (m.stride > 0 && lg_strided(m, lg_div_b(m, j))));
    if (live != lg_live(m, i, j)) return 6;
  }
  return 0;
}
"""


def run(tmp_path, program, opt):
    src, exe = tmp_path / "program.cpp", tmp_path / "program"
    src.write_text(program)
    subprocess.check_call(["g++", "-std=c++17", opt, "-I", CSRC, str(src), "-o", str(exe)])
    r = subprocess.run([str(exe)], stdout=subprocess.PIPE, text=True)
    assert r.returncode == 0, (r.returncode, r.stdout)


def test_classes_and_runs_from_bounds(tmp_path):
    run(tmp_path, KINDS, "-O2")


@pytest.mark.parametrize("opt", ["-O0", "-O2"])
def test_runs_cover_every_item_once_and_give_the_xcds_even_shares(tmp_path, opt):
    """Where rows grow and heads are few: with runs of 16 tiles listed head by head an XCD had up to twice its share."""
    run(tmp_path, RUNS, opt)


def test_engines_and_cus_get_even_shares(tmp_path):
    """With two heads in four the other way round the CUs of launches of one or two rounds got up to 1.5 times their share; with
    four heads side by side launches of many rounds lost up to 7 % to keys that an L2 does not hold."""
    run(tmp_path, ORDER, "-O2")


@pytest.mark.parametrize("opt", ["-O0", "-O2"])
def test_division_by_multiplication_and_items(tmp_path, opt):
    run(tmp_path, PROGRAM, opt)


LISTS = r"""
#include <cstdio>
#include "lg_mask.h"
// N, sink, window, block, stride, and whether tiles are listed: causal rows of 9 and 10 tiles, windows, columns near and far
int main() {
  const int shapes[][6] = {{1, 0, 1, 1, 0, 0}, {576, 0, 576, 1, 0, 0}, {577, 0, 577, 1, 0, 1}, {9000, 0, 9000, 1, 0, 1}, {9000, 64, 384, 64, 0, 0},
                           {9088, 64, 448, 64, 0, 0}, {9088, 64, 512, 64, 0, 1}, {9088, 64, 64, 64, 0, 0}, {24000, 64, 64, 64, 16, 1}, {24000, 64, 64, 64, 17, 0}, {24000, 64, 64, 64, 64, 0},
                           {24000, 64, 640, 64, 64, 0}, {24000, 128, 128, 128, 16, 1}, {24000, 16, 64, 16, 64, 1}, {24000, 16, 64, 16, 65, 0},
                           {24000, 0, 64, 1, 1024, 1}, {24000, 0, 64, 1, 1025, 0}, {600, 64, 64, 64, 8, 0}, {130, 0, 130, 1, 0, 0}};
  for (auto& s : shapes)
    if (lg_fwd_lists(lg_make_mask(s[0], s[1], s[2], s[3], s[4]), 128) != (s[5] != 0)) { std::printf("%d %d %d %d %d\n", s[0], s[1], s[2], s[3], s[4]); return 1; }
  return 0;
}
"""


def test_which_small_forwards_list_their_tiles(tmp_path):
    """Rows of a few tiles, and tiles that are live few and far between, are walked without a list."""
    run(tmp_path, LISTS, "-O1")


SHARED = r"""
#include <cstdio>
#include <vector>
#include "lg_mask.h"
// B x heads, N, window, tile: dk/dv's items beside dq's, as the hardware deals them
int main() {
  const int shapes[][4] = {{4, 16384, 16384, 256}, {2, 48000, 48000, 256}, {3, 13989, 4663, 256}, {1, 65000, 65000, 256}, {4, 24000, 24000, 256},
                           {9, 4096, 4096, 128}, {6, 5666, 1888, 128}, {8, 6000, 6000, 256}, {12, 5218, 5218, 128}, {5, 6000, 6000, 256}};
  for (auto& s : shapes) {
    const int heads = s[0], N = s[1], TK = s[3], tiles = (N + TK - 1) / TK, total = tiles * heads;
    const LgMask m = lg_make_mask(N, 0, s[2], 1, 0);
    const bool by_tile = lg_dkdv_by_tile(m, heads, total, true);
    const int run = lg_run_length(m, total, heads, 8, false);
    const long long grid = by_tile ? total : lg_run_grid(total, run);
    std::vector<int> seen(total, 0);
    double work[8] = {}, all = 0, longest = 0;
    for (long long id = 0; id < grid; ++id) {
      const int L = by_tile ? (int)(id % heads * tiles + id / heads) : lg_item_of((int)id, run);
      if (L >= total) continue;
      ++seen[L];
      const int k0 = L % tiles * TK, last = k0 + TK - 1 + s[2] - 1, end = last < N - 1 ? last : N - 1;
      const double steps = 4 + end / 64 - k0 / 64;
      work[id & 7] += steps;
      all += steps;
      longest = steps > longest ? steps : longest;
    }
    for (int x : seen)
      if (x != 1) return 2;
    for (double x : work)
      if (x > 1.1 * all / 8 + longest) { std::printf("%d heads, %d tokens: an XCD has %.0f of %.0f steps\n", heads, N, x, all / 8); return 3; }
  }
  return 0;
}
"""


def test_dkdv_beside_dq_gives_the_xcds_even_shares(tmp_path):
    """In runs of 8 tiles one XCD had the longest tiles of all of 4 heads of 64 tiles."""
    run(tmp_path, SHARED, "-O2")
