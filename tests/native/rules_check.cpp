// CPU check of the rules that choose kernels and tile widths (sht_plan.h).
// Built and run by tests/test_host_rules.py.
#include <algorithm>
#include <cstdio>
#include <map>
#include <numeric>
#include <tuple>
#include <vector>

#include "sht_plan.h"
#include "sht_zonal_rule.h"

using namespace sht;

static int g_fail = 0;
#define CHECK(c, ...)                                                     \
  do {                                                                    \
    if (!(c)) {                                                           \
      std::printf("check failed: %s (line %d): ", #c, __LINE__);          \
      std::printf(__VA_ARGS__);                                           \
      std::printf("\n");                                                  \
      ++g_fail;                                                           \
    }                                                                     \
  } while (0)

constexpr int kCu = 256;

// the width a plan takes for one direction
static int width(int form, bool gen, bool analysis, int N, int J, int F) {
  const int FB = zonal_fields_per_block(form);
  const int g = choose_granularity(form, gen, 1, &N, &J, &F, FB, kCu, SHT_NOALLOC_WORKSPACE_BYTES);
  const long long Cp = roundup(2LL * F, std::lcm(16LL * g, 2LL * FB));
  const std::vector<int> jst(N + 1, 0);
  const int def = default_tile(form, 1, &N, &J, &F, FB, jst.data(), analysis, kCu);
  return choose_tile(form, gen, 1, &N, &J, &F, &Cp, jst.data(), analysis, def, kCu, nullptr);
}

// Shapes where the estimate alone picked a width that measured slower than
// the one expected here (us in the comments: expected, the estimate's), and
// shapes where another width than the default's is worth far more than the
// margin.
static void check_widths() {
  struct {
    int form;
    bool gen, analysis;
    int N, J, F, expect;
  } const rows[] = {
      {SHT_FORM_FP64, true, false, 213, 214, 48, 2},    // 33.3, 45.9 with 3
      {SHT_FORM_FP64, true, false, 213, 427, 48, 2},    // 54, 67.5 with 6
      {SHT_FORM_FP64, true, false, 639, 1279, 48, 6},   // 650, 766 with 3
      {SHT_FORM_FP64, true, false, 720, 33, 48, 2},     // 125, 173 with 3
      {SHT_FORM_FP32, true, true, 255, 511, 200, 5},    // 147, 203.5 with 7
      {SHT_FORM_FP32, true, true, 426, 853, 200, 5},    // 510, 703.9 with 7
      {SHT_FORM_FP32, false, true, 341, 683, 48, 2},    // 60, 71.9 with 6
      {SHT_FORM_FP32, false, true, 159, 160, 72, 1},    // 14.7, 16.9 with 9
      {SHT_FORM_FP64, false, true, 106, 213, 400, 2},   // 64, 77.5 with 8
      {SHT_FORM_FP64, false, true, 319, 320, 16, 2},    // 26, 31.1 with 1
      {SHT_FORM_FP64, false, true, 170, 341, 19, 3},    // 17.6, 18.4 with 1
      {SHT_FORM_FP64, false, true, 63, 127, 64, 2},     // 8.0, 8.7 with 3
      {SHT_FORM_FP64, false, false, 159, 160, 128, 4},  // 37, 44.4 with 2
      {SHT_FORM_FP64, false, false, 341, 342, 32, 4},   // 67, 78.6 with 2
      {SHT_FORM_FP32, false, true, 479, 959, 100, 7},   // 264, 345 with the default's 1
      {SHT_FORM_FP32, false, false, 479, 959, 100, 7},  // 278, 443
      {SHT_FORM_BF16X6, false, false, 319, 639, 45, 6}, // 59, 93
  };
  for (const auto& r : rows) {
    const int k = width(r.form, r.gen, r.analysis, r.N, r.J, r.F);
    CHECK(k == r.expect, "form %d gen %d analysis %d N %d J %d F %d: %d, expected %d", r.form, r.gen, r.analysis, r.N,
          r.J, r.F, k, r.expect);
  }
  // no width that spills, at any field count
  for (int F = 1; F <= 400; ++F) {
    const int k = width(SHT_FORM_FP32, true, true, 300, 601, F);
    CHECK(k != 7 && k != 9, "F %d: %d", F, k);
  }
}

// The autotuner times the width a plan has without it, also where its tiles
// are fewer than the compute units, and every width of the least-padding rule.
static void check_tune_widths() {
  auto has = [](const std::vector<int>& w, int k) {
    for (int x : w)
      if (x == k) return true;
    return false;
  };
  for (int form : {SHT_FORM_FP64, SHT_FORM_FP32, SHT_FORM_BF16X6})
    for (int N : {21, 80, 106, 170, 319})
      for (int F = 1; F <= 130; ++F)
        for (int dir = 0; dir < 2; ++dir) {
          const int J = 2 * N + 1, FB = zonal_fields_per_block(form);
          const int g = choose_granularity(form, false, 1, &N, &J, &F, FB, kCu, SHT_NOALLOC_WORKSPACE_BYTES);
          const long long Cp = roundup(2LL * F, std::lcm(16LL * g, 2LL * FB));
          const std::vector<int> jst(N + 1, 0);
          const int def = default_tile(form, 1, &N, &J, &F, FB, jst.data(), dir == 0, kCu);
          const std::vector<int> w = tune_widths(form, false, 1, &N, &J, &F, &Cp, jst.data(), dir == 0, def, kCu);
          CHECK(has(w, width(form, false, dir == 0, N, J, F)), "form %d N %d F %d dir %d", form, N, F, dir);
          for (int k : {1, 2, 4, 5, 8, 10})
            CHECK(has(w, k) == (k <= max_ncb(form, dir == 0) && Cp % (16 * k) == 0), "form %d N %d F %d dir %d: %d", form,
                  N, F, dir, k);
        }
}

// A cached line is one plan's: the key tells apart the kernels it was timed
// on, the reduced transform and the grid (other tile lists).
static void check_tune_key() {
  const int N = 170, J = 341, I = 512, F = 19;
  LevelDesc lev[SHT_MAX_LEVELS];
  Layout Y;
  layout_levels(1, &N, &J, &I, &F, 48, 4, lev, &Y);
  const std::string k = tune_plan_key(SHT_FORM_FP64, 4, SHT_GRID_FEJER2, false, 1, lev);
  CHECK(k != tune_plan_key(SHT_FORM_FP64, 4, SHT_GRID_FEJER2, true, 1, lev), "reduced: %s", k.c_str());
  CHECK(k != tune_plan_key(SHT_FORM_FP64, 4, SHT_GRID_GAUSS, false, 1, lev), "grid: %s", k.c_str());
  // the key of the lines timed on the kernels before the present ones
  CHECK(k.find("v3 form") == std::string::npos && k.find("v3 kern") == 0, "generation: %s", k.c_str());
}

static LevelDesc level(int J, int I, int F) {
  LevelDesc L{};
  L.N = I / 3;
  L.J = J;
  L.Jh = (J + 1) / 2;
  L.I = I;
  L.F = F;
  return L;
}

// The group kernels take levels with few items (fewer than compute units),
// whose empty sequences cost nothing, and leave mostly empty groups to the
// any-length kernels only where every unit has an item.  Times in us: group,
// any-length.
static void check_group_rule() {
  struct {
    bool dbl, analysis;
    int J, I, F;
    bool takes;
  } const rows[] = {
      {true, true, 479, 960, 3, true},     // 14, 18: the Tl479 grid of the aliasing experiment
      {true, false, 479, 960, 3, true},    // 14, 18
      {true, true, 64, 1600, 20, true},    // 18, 24
      {false, false, 64, 400, 8, true},    // 8, 11
      {false, false, 427, 480, 1, true},   // 9, 13
      {true, false, 64, 400, 1, true},     // 7, 9
      {false, true, 641, 1920, 1, false},  // 22, 16
      {true, true, 641, 1600, 1, false},   // 21, 16
      {false, true, 641, 1440, 64, true},  // many full groups
  };
  for (const auto& r : rows) {
    const int fc = group_fields(r.dbl, r.analysis, r.I);
    CHECK(fc >= 1 && fc <= 8, "I %d: %d", r.I, fc);
    CHECK(group_takes(fc, level(r.J, r.I, r.F), kCu) == r.takes, "dbl %d analysis %d J %d I %d F %d", r.dbl, r.analysis,
          r.J, r.I, r.F);
  }
  CHECK(group_fields(false, true, 256) == 0 && group_fields(true, true, 1000) == 0, "lengths without a group kernel");
  CHECK(level_shares(false, true, level(129, 200, 3), kCu), "no group kernel");
  CHECK(level_shares(false, true, level(257, 400, 3), kCu), "few items");
  CHECK(level_shares(false, true, level(641, 960, 1), kCu), "mostly empty groups");
  CHECK(!level_shares(false, true, level(1025, 1600, 32), kCu), "many items");
}

// The register-held kernels take full, large levels only.  Times in us: group,
// held.
static void check_held_rule() {
  struct {
    bool dbl;
    int N, J, I, F, Cp;
    bool takes;
  } const rows[] = {
      {false, 959, 1919, 2880, 64, 128, true},    // 710, 579
      {false, 959, 1919, 2880, 32, 64, true},     // 313, 300
      {false, 1023, 2049, 3072, 64, 128, true},   // 847, 634
      {false, 719, 641, 2160, 1, 16, false},      // one field of eight, 1.9 times as long
      {false, 960, 641, 2880, 8, 16, false},      // 37, 52
      {false, 1024, 128, 3072, 128, 256, true},   // 119, 109
      {false, 719, 641, 2160, 64, 128, false},    // 1.12 times as long
      {false, 799, 641, 2400, 96, 192, false},    // 1.06
      {false, 767, 33, 2304, 64, 128, false},     // 1.13
      {true, 959, 1919, 2880, 64, 128, true},     // 1473, 1164
      {true, 767, 128, 2304, 64, 128, true},      // 79, 67
      {true, 1439, 641, 2880, 64, 128, true},     // 659, 581
      {true, 1439, 641, 2880, 12, 32, false},     // 94, 118
      {true, 1079, 641, 2160, 128, 256, false},   // 832, 983
      {true, 1023, 2049, 3072, 64, 128, false},   // 1745, 1697: spills
      {true, 959, 33, 2880, 64, 128, false},      // 1.26
  };
  for (const auto& r : rows) {
    LevelDesc L = level(r.J, r.I, r.F);
    L.N = r.N;
    L.Cp = r.Cp;
    CHECK(held_takes(r.dbl, L) == r.takes, "dbl %d N %d J %d I %d F %d", r.dbl, r.N, r.J, r.I, r.F);
  }
}

// One launch over all levels by default (I = 100 2^k, J = 64 2^k + 1): FP64
// plans of few fields, which took it before the group kernels (five levels, 3
// fields, synthesis 45 us against 58 per length).
static void check_one_launch() {
  auto def = [](bool dbl, bool analysis, int nlev, int F) {
    LevelDesc lev[SHT_MAX_LEVELS];
    for (int l = 0; l < nlev; ++l) lev[l] = level((64 << l) + 1, 100 << l, F);
    return one_launch_default(dbl, analysis, nlev, lev, kCu);
  };
  for (int ana = 0; ana < 2; ++ana) {
    for (int F : {3, 5, 8}) CHECK(def(true, ana, 5, F) && def(true, ana, 4, F), "analysis %d F %d", ana, F);
    CHECK(!def(true, ana, 5, 1) && !def(true, ana, 5, 32) && !def(true, ana, 3, 3) && !def(true, ana, 1, 3),
          "analysis %d", ana);
    for (int F : {1, 3, 8, 32}) CHECK(!def(false, ana, 5, F), "analysis %d F %d", ana, F);
  }
}

// Tile lists of the widths that no power of two gives: every (m, row or
// latitude block, column block) once, nothing else, in both orders, with and
// without latitudes left out.  (Built with the planner's bounds assertions.)
static void check_odd_tiles() {
  struct {
    int form, N, J, I, F;
  } const plans[] = {{SHT_FORM_FP64, 130, 261, 300, 21}, {SHT_FORM_FP32, 140, 101, 288, 67},
                     {SHT_FORM_FP32, 40, 300, 96, 103},  {SHT_FORM_BF16X6, 300, 97, 640, 45}};
  for (const auto& c : plans)
    for (int k : {3, 6, 7, 9})
      for (int part = 0; part < 2; ++part) {
        LevelDesc lev[SHT_MAX_LEVELS];
        Layout Y;
        layout_levels(1, &c.N, &c.J, &c.I, &c.F, 16 * k, zonal_fields_per_block(c.form), lev, &Y);
        std::vector<int> jst(Y.nm_total, 0);
        for (int m = 0; part && m < Y.nm_total; ++m) jst[m] = std::min(32 * (m % 5), lev[0].Jh);
        for (int dir = 0; dir < 2; ++dir)
          for (int sched = 0; sched < 2 && k <= max_ncb(c.form, dir == 0); ++sched) {
            std::map<std::tuple<int, int, int>, int> seen;
            for (const Tile& t : build_tiles(c.form, 1, lev, jst.data(), dir == 0, k, sched))
              if (t.level >= 0) seen[{t.m, t.rb, t.cb}] += 1;
            size_t n = 0;
            const int rows = c.form == SHT_FORM_BF16X6 ? 256 : 128;
            for (int m = 0; m <= c.N; ++m)
              for (int cb = 0; 16 * k * cb < 2 * c.F; ++cb)
                for (int b = dir == 0 ? 0 : jst[m] / 128;
                     dir == 0 ? b * rows < c.N - m + 1 : b * 128 < lev[0].Jh; ++b, ++n)
                  CHECK(seen[std::make_tuple(m, b, cb)] == 1, "form %d k %d dir %d m %d block %d column %d", c.form, k,
                        dir, m, b, cb);
            CHECK(seen.size() == n, "form %d k %d dir %d", c.form, k, dir);
          }
      }
}

// The any-length kernels' shapes: what an item holds fits its threads and the
// LDS, and the vectors of a row cover it and stay in it, for every length that
// a plan takes and the largest wavenumber it may have.
static void check_any_shapes() {
  for (size_t size : {4, 8}) {
    const int E = any_values(size), V = 16 / (int)size;
    for (int I = 1; I <= 4096; ++I) {
      int rad[SHT_MAX_RADICES], nrad = 0;
      if (!factor_radices(I, rad, &nrad)) continue;
      for (int F : {1, 2, 3, 64})
        for (int J : {3, 641}) {
          LevelDesc L = level(J, I, F);
          L.N = (I - 1) / 2;
          L.nrad = nrad;
          std::copy(rad, rad + nrad, L.rad);
          if (((size_t)any_stride(L) + 1 + I) * 2 * size > kAnyMaxLds || I > 512 * E) continue;
          const AnyShape s = any_choice(size, 1, &L, kCu);
          const long long fc = 1 << s.lfc, rows = s.vec ? (I + V - 1) / V * V : I;
          CHECK(s.nt == 256 || s.nt == 512 || (s.nt == 1024 && size == 4 && s.lfc == 1 && s.vec),
                "%zu I %d F %d: %d threads", size, I, F, s.nt);
          CHECK(fc * rows <= (long long)s.nt * E && 2 * fc * (L.N + 1) <= (long long)s.nt * E &&
                    fc * any_stride(L) <= s.tw_lds && s.lds <= kAnyMaxLds &&
                    (s.tw_lds + (size_t)I) * 2 * size <= s.lds,
                "%zu I %d F %d J %d: %lld fields, %d threads, %zu bytes", size, I, F, J, fc, s.nt, s.lds);
          CHECK(s.vec == (I >= V), "%zu I %d", size, I);
        }
    }
    for (int I = V; I < 700; ++I) {
      std::vector<int> seen(I, 0);
      const int nv = size == 4 ? any_nvec<4>(I) : any_nvec<2>(I);
      for (int v = 0; v < nv; ++v) {
        const int i = size == 4 ? any_first<4>(v, I) : any_first<2>(v, I);
        CHECK(i >= 0 && i + V <= I, "%zu I %d vector %d", size, I, v);
        for (int e = 0; e < V; ++e) seen.at(i + e) += 1;
      }
      CHECK(*std::min_element(seen.begin(), seen.end()) >= 1, "%zu I %d", size, I);
    }
  }
  struct {
    size_t size;
    int I, F, fields, threads;
  } const rows[] = {
      {4, 625, 64, 8, 512},   // odd rows in vectors too
      {4, 3375, 64, 2, 1024}, {4, 3375, 1, 1, 512}, {4, 3000, 64, 2, 512},
      {8, 625, 64, 2, 256},   {8, 810, 64, 2, 256}, {8, 1080, 64, 2, 512},
  };
  for (const auto& r : rows) {
    LevelDesc L = level(641, r.I, r.F);
    CHECK(factor_radices(r.I, L.rad, &L.nrad), "%d", r.I);
    const AnyShape s = any_choice(r.size, 1, &L, kCu);
    CHECK(1 << s.lfc == r.fields && s.nt == r.threads && s.vec, "%zu I %d F %d: %d fields, %d threads", r.size, r.I,
          r.F, 1 << s.lfc, s.nt);
  }
}

int main() {
  check_any_shapes();
  check_odd_tiles();
  check_widths();
  check_one_launch();
  check_held_rule();
  check_group_rule();
  check_tune_widths();
  check_tune_key();
  std::printf("rules_check: %d failures\n", g_fail);
  return g_fail ? 1 : 0;
}
