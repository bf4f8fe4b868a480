// Host-side layout planning of the transform library: the per-level sizes
// and offsets of the tables, seed rows and workspace, the tile lists of the
// Legendre kernels, and the filling of the blocked table copies.  Plain C++
// (no HIP), so that it is built into the library and, with bounds
// assertions (SHT_CHECK) and sanitizers, into a CPU check.
#ifndef SHT_PLAN_H_
#define SHT_PLAN_H_

#include <string>
#include <vector>

#include "sht_internal.h"

#ifdef SHT_CHECK
#include <cstdio>
#include <cstdlib>
#define SHT_ASSERT(c)                                                                   \
  do {                                                                                  \
    if (!(c)) {                                                                         \
      std::fprintf(stderr, "SHT_CHECK failed: %s (%s:%d)\n", #c, __FILE__, __LINE__); \
      std::abort();                                                                     \
    }                                                                                   \
  } while (0)
#else
#define SHT_ASSERT(c) ((void)0)
#endif

namespace sht {

inline long long roundup(long long a, long long b) { return (a + b - 1) / b * b; }

// Time estimate of one direction's Legendre kernel with column tiles of k
// 16-column blocks on ncu compute units, in units of one K block's products
// for one column block: every tile costs (K blocks) (k + a) with a the work
// of a K block that does not depend on the tile's width.  a was fitted, with
// the shape of the sum over tiles, to timings of every width at truncations
// 21..639 with J = 2N + 1 and N + 1 and 8..400 fields (1000 plans with tables,
// 1245 with generated P~); the widths it picks take 1.00 to 1.05 times the
// best one's time (geometric mean per form and direction).
// gen: generated P~; jst as for build_tiles (or null).
double legendre_cost(int form, bool gen, int nlev, const int* N, const int* J, const int* F, const int* jst,
                     bool analysis, int k, int ncu);

// The width a direction takes unless the estimate promises more: of the
// widths 1, 2, 4, 5, 8, 10 the one that pads the columns least (the wider on
// ties), narrowed as long as the compute units would get fewer than two tiles
// each.
int default_tile(int form, int nlev, const int* N, const int* J, const int* F, int FB, const int* jst, bool analysis,
                 int ncu);

// Whether tiles of k column blocks cover every level's workspace row exactly.
bool width_tiles(int nlev, const long long* Cp, int k);

// Column blocking of a direction: of the widths that tile every level's
// workspace row Cp exactly the one of least estimated time, where a width
// other than def (default_tile) has to gain 5 %, about what the estimate can
// tell apart.  Over the 4500 kernels of the fit the estimate alone took more
// than 3 % longer than def in 220, the worst 38 % (FP64 with generated P~,
// N = 213, 48 fields, synthesis: 45.9 us with three blocks, 33.4 with def's
// two); with the margin in 42, the worst 17 %.
int choose_tile(int form, bool gen, int nlev, const int* N, const int* J, const int* F, const long long* Cp,
                const int* jst, bool analysis, int def, int ncu, double* cost);

// The widths the autotuner times for a direction, of those that tile the
// rows: the plan's own (def and the one choose_tile takes), 1, 2, 4, 5, 8 and
// 10, and the others where the estimate lies within a quarter of the least.
// (Whether a width leaves compute units without a tile says nothing: FP64,
// T170 with 19 fields, analysis, 214 tiles of three blocks 17.6 us, 642 of one
// 17.8.  The widths left out are the best ones by more than 2 % in 8 of 2100
// timed kernels, by 9 % at most.)
std::vector<int> tune_widths(int form, bool gen, int nlev, const int* N, const int* J, const int* F,
                             const long long* Cp, const int* jst, bool analysis, int def, int ncu);

// The part of the tuner's cache key that does not depend on the device: line
// format v3, the generation of the kernels that were timed (kKernelGen: raised
// whenever Legendre or zonal kernels or the candidates change, so that a line
// timed on others is not used), form, zonal item width, grid and reduced
// transform (which fix the latitudes left out, so the tile lists), and every
// level's sizes and row length.
constexpr int kKernelGen = 2;
std::string tune_plan_key(int form, int fb, int grid, bool reduced, int nlev, const LevelDesc* lev);

// Granularity g of the workspace rows (16-column blocks; Cp is 2 F rounded
// up to lcm(16 g, 2 FB)): the one whose divisors serve both directions best.
// 100 fields (13 blocks) take 14 blocks, two tiles of 7: Legendre analysis /
// synthesis at T479 FP32 0.264 / 0.278 ms, against 0.345 / 0.443 with 13
// tiles of one block, which pads least.  Rows that would lift the workspace
// over ws_limit bytes are not considered where tighter ones stay below it.
int choose_granularity(int form, bool gen, int nlev, const int* N, const int* J, const int* F, int FB, int ncu,
                       long long ws_limit);
// The same for items of the default width, table kernels and a whole device.
int choose_ncb(int form, int nlev, const int* N, const int* J, const int* F);

// Offsets of one plan's per-(level, m) blocks and its totals (elements);
// each offset vector has one sentinel entry past the last (level, m).
struct Layout {
  std::vector<long long> taboff;      // analysis table copy
  std::vector<long long> taboff_syn;  // synthesis table copy
  std::vector<long long> seedoff;     // seed rows of generated P~
  std::vector<long long> recoff;      // recurrence coefficients
  long long tab = 0, tabs = 0, seeds = 0, rec = 0;
  long long items = 0;                // zonal work items
  long long grid = 0, spec = 0, ws = 0;
  int nm_total = 0;                   // (level, m) pairs
};

// Fill the level descriptors (sizes, FFT radices, offsets; the device
// pointers stay null) for column tiles of BN columns and zonal items of FB
// fields, and the offsets of every (level, m) block.
void layout_levels(int nlev, const int* N, const int* J, const int* I, const int* F, int BN, int FB,
                   LevelDesc* lev, Layout* out);

// Tile list of one Legendre kernel for column blocking ncb (16*ncb columns
// per tile; every level's workspace row length Cp must be a multiple of it).
// jst: per (level, m) first latitude kept (reduced transform; else 0).
// sched 0: locality order (m, column block, row block) cut into 8 chunks of
// equal cost, chunk x dealt to block ids == x (mod 8), i.e. to XCD x;
// sched 1: the same order dealt round robin.
std::vector<Tile> build_tiles(int form, int nlev, const LevelDesc* lev, const int* jst, bool analysis, int ncb,
                              int sched);

// Fill both blocked copies of one level's table (dst / dsyn may be null:
// then only j0 and seeds are produced) from FP64 columns of P~; j0 (may be
// null): per m the first latitude with some |P~_n^m| >= 1e-16; seeds (may be
// null): rows 16 g and 16 g + 1 of every 16-degree group g, Kp long.  The
// per-m offsets are those of layout_levels.
template <typename T>
void fill_table_level(const LevelDesc& L, const double* mu, const double* sint, T* dst, const long long* off_a,
                      T* dsyn, const long long* off_s, int* j0, double* seeds, const long long* off_seed);

}  // namespace sht

#endif  // SHT_PLAN_H_
