// Which zonal kernel a level takes: the lengths, shapes and choices of the
// group kernels (sht_group.h), the any-length ones (sht_any.h) and the
// register-held ones (sht_fft.hip).
// Plain C++ (no HIP), so that the rules are checked on the CPU too.
#ifndef SHT_ZONAL_RULE_H_
#define SHT_ZONAL_RULE_H_

#include "sht_internal.h"

namespace sht {

// Every length 16 R2 R3 from 288 on with radices up to 16.
#define SHT_GROUP_LENGTHS(X)                                                                                      \
  X(288) X(320) X(384) X(400) X(432) X(480) X(512) X(576) X(640) X(720) X(768) X(800) X(864) X(960) X(1024)       \
  X(1152) X(1200) X(1280) X(1296) X(1440) X(1536) X(1600) X(1728) X(1920) X(2048) X(2160) X(2304) X(2400) X(2560) \
  X(2880) X(3072) X(3600) X(3840) X(4096)

// Radices of the second and third pass for NT threads and FC sequences: a
// thread holds ceil(FC (I / R) / NT) butterflies of R values in a pass; the
// pair of least sum (a second, nearly empty round of butterflies costs as
// much as a full one, and its registers), then the larger second radix.
constexpr bool grp_radix(int r) {
  return r == 2 || r == 3 || r == 4 || r == 5 || r == 6 || r == 8 || r == 9 || r == 10 || r == 12 || r == 15 || r == 16;
}
constexpr int grp_held(int I, int R, int NT, int FC) { return (FC * (I / R) + NT - 1) / NT * R; }
constexpr int grp_r2(int I, int NT, int FC) {
  int best = 0, cost = 1 << 30;
  for (int r = 16; r >= 2; --r) {
    const int q = I / 16;
    if (q % r || !grp_radix(r) || !grp_radix(q / r)) continue;
    const int c = grp_held(I, r, NT, FC) + grp_held(I, q / r, NT, FC);
    if (c < cost) {
      cost = c;
      best = r;
    }
  }
  return best;
}
constexpr int grp_most_held(int I, int NT, int FC) {
  const int r2 = grp_r2(I, NT, FC), a = grp_held(I, r2, NT, FC), b = grp_held(I, I / 16 / r2, NT, FC);
  return a > b ? a : b;
}

// Three passes of radices 16, R2, R3 over sequences that lie side by side in
// LDS.  The first pass stores element 16 j + t at the padded position
// 17 j + t, so that the lanes of a wave, which own consecutive j, hit
// distinct banks; the second reads that order (its inputs j + t I/R2 sit at
// j + j/16 + t (17/16)(I/R2), I/R2 being a multiple of 16) and writes the
// natural order; the third reads and writes the natural order.  Twiddles of
// passes two and three are staged in LDS as [t-1][k] (k = butterfly position
// within its Ns-block).
template <int I_, int R2_, int R3_>
struct Plan3 {
  static constexpr int I = I_, R1 = 16, R2 = R2_, R3 = R3_;
  static_assert(R1 * R2 * R3 == I, "radices must multiply to I");
  static constexpr int nb1 = I / R1, nb2 = I / R2, nb3 = I / R3;
  static constexpr int Ns2 = R1, Ns3 = R1 * R2;
  static_assert(nb3 == Ns3, "last pass");
  static_assert(I % 16 == 0 && nb2 % 16 == 0, "padded layout");
  static constexpr int IP = I + I / 16;        // padded field stride
  static constexpr int S2P = nb2 + nb2 / 16;   // padded stride of pass-2 inputs
  static constexpr int tw2 = 0, tw3 = (R2 - 1) * Ns2, ntw = tw3 + (R3 - 1) * Ns3;
};

// Shape of a length's kernel: NT threads, FC fields per item, waves per SIMD
// the registers are sized for, PF: the next item is fetched into registers
// during the current one (else another workgroup covers the latency).
// Chosen from sweeps over lengths (MI355X, 801 or 1601 rows, analysis /
// synthesis in us; "held" = the kernels of sht_fft.hip where they exist, else
// those of sht_any.h):
//  FP32, 300 fields      480: 72 / 66 (held 87 / 74)       1024: 310 / 281 (413 / 424)
//                        800: 202 / 171 (236 / 263)        1280: 476 / 487 (603 / 626)
//  FP32, 400 fields 1440: 852 / 900 (1045 / 1061)   64 fields 2048: 279 / 300 (445 / 453)
//  FP64, 48 fields       640: 40 / 39 (78 / 78)            1280: 152 / 149 (272 / 318)
// FP32 analysis takes all 8 fields of a workspace block (64-byte pieces;
// with 4 fields 1440 rose to 1137) while a thread holds at most 16 values
// and a pass at most 20 per buffer; FP32 synthesis mostly 4.  From 1600 on
// one workgroup fills a compute unit's LDS: it has 1024 threads and fetches
// ahead.  Five of the 136 kernels spill: FP32 synthesis 1296, 1600 and 3600 (2,
// 9 and 19 registers), FP64 analysis 1600 and 1728 (30 and 29).
template <typename T, int I, bool ANA>
struct GroupShape {
  static constexpr bool dbl = sizeof(T) == 8;
  static constexpr bool all8 =
      !dbl && (ANA ? I <= 2048 && grp_most_held(I, I <= 512 ? 256 : I <= 1024 ? 512 : 1024, 8) <= 20
                   : I > 512 && I <= 1024 && grp_most_held(I, 512, 8) <= 16);
  static constexpr int NT = dbl ? (I <= 1024 ? 256 : 512)
                            : all8 ? (I <= 512 ? 256 : I <= 1024 ? 512 : 1024)
                                   : (I <= 512 ? 256 : I <= 1600 ? 512 : 1024);
  static constexpr int FC = dbl ? (I <= 1920 ? 4 : I <= 3072 ? 2 : 1) : all8 ? 8 : I <= 3840 ? 4 : 2;
  static constexpr bool PF = dbl ? (I > 1024 && (ANA || I <= 1280 || I > 1920)) : !all8 && I > 1600;
  static constexpr int WPE = dbl ? 2 : 4;
  using P = Plan3<I, grp_r2(I, NT, FC), I / 16 / grp_r2(I, NT, FC)>;
};

// Fields per item of a length's group kernel; 0 where there is none.
inline int group_fields(bool dbl, bool analysis, int I) {
  switch (I) {
#define SHT_GROUP_FIELDS(i)                                                                         \
  case i:                                                                                           \
    return dbl ? (analysis ? GroupShape<double, i, true>::FC : GroupShape<double, i, false>::FC)    \
               : (analysis ? GroupShape<float, i, true>::FC : GroupShape<float, i, false>::FC);
    SHT_GROUP_LENGTHS(SHT_GROUP_FIELDS)
#undef SHT_GROUP_FIELDS
    default: return 0;
  }
}

// The any-length kernels (sht_any.h): complex values per thread, so that
// FC I <= NT E (I in whole vectors) and FC (N + 1) <= NT E / 2; the LDS of a
// workgroup.
constexpr int any_values(size_t value_size) { return value_size == 4 ? 12 : 8; }
constexpr size_t kAnyMaxLds = 160 * 1024;

// Field stride in LDS: room for the padded first pass; 2 mod 16, so that
// the fold's lanes (adjacent wavenumbers of several fields) spread over the
// banks.
constexpr int any_stride(const LevelDesc& L) {
  const int pad = L.nrad > 1 && L.rad[0] % 2 == 0 ? L.I / L.rad[0] : 0;
  return ((L.I + pad + 15) & ~15) + 2;
}

// Vectors of a row, and the first value of vector v.
template <int V>
constexpr int any_nvec(int I) {
  return (I + V - 1) / V;
}
template <int V>
constexpr int any_first(int v, int I) {
  return V == 1 || v * V < I - V ? v * V : I - V;
}

struct AnyShape {
  int lfc, nt;  // log2 of the fields per item, threads per item
  bool vec;     // rows as 16-byte vectors
  int tw_lds;   // LDS offset of the twiddles, complex values
  size_t lds;   // bytes
};

inline AnyShape any_choice(size_t value_size, int nlev, const LevelDesc* lev, int ncu) {
  const int E = any_values(value_size), V = 16 / (int)value_size;
  int maxI = 0, maxR = 0, maxN = 0, maxIP = 0, maxF = 0;  // maxR: whole vectors
  bool vec = true;
  for (int l = 0; l < nlev; ++l) {
    const LevelDesc& L = lev[l];
    maxI = L.I > maxI ? L.I : maxI;
    maxN = L.N > maxN ? L.N : maxN;
    maxF = L.F > maxF ? L.F : maxF;
    const int ip = any_stride(L);
    maxIP = ip > maxIP ? ip : maxIP;
    const int r = (L.I + V - 1) / V * V;
    maxR = r > maxR ? r : maxR;
    vec = vec && L.I >= V;
  }
  // fields per item: as many as a workspace run holds, as long as two
  // workgroups share a compute unit's LDS, no group is mostly empty and the
  // device has an item per compute unit (T85 with 7 fields: 28 us a pair with
  // two per unit, one field each, 24 with one)
  auto tw_of = [&](int fc) { return (fc * maxIP + 1) & ~1; };
  auto lds_of = [&](int fc) { return ((size_t)tw_of(fc) + maxI) * 2 * value_size; };
  auto items_of = [&](int fc) {
    long long n = 0;
    for (int l = 0; l < nlev; ++l) n += (long long)lev[l].Jh * ((lev[l].F + fc - 1) / fc);
    return n;
  };
  auto holds = [&](int fc, long long nt) { return fc * (long long)maxR <= nt * E && fc * (maxN + 1LL) <= nt / 2 * E; };
  int lfc = value_size == 4 ? 3 : 2;
  while (lfc > 0 && (!holds(1 << lfc, 512) || lds_of(1 << lfc) > kAnyMaxLds / 2 || (1 << (lfc - 1)) >= maxF ||
                     items_of(1 << lfc) < ncu))
    --lfc;
  // FP64 at 512 to 1024: groups that 256 threads hold, so that two workgroups
  // share a compute unit (641 rows, 64 fields, analysis / synthesis: 625 101 /
  // 95 -> 87 / 84 us, 810 152 / 131 -> 138 / 130; longer rows lose up to 12 %)
  if (value_size == 8 && maxR > 512 && maxR <= 1024)
    while (lfc > 0 && !holds(1 << lfc, 256)) --lfc;
  // FP32 rows of which 512 threads hold one field: 1024 threads hold two, whose
  // workspace pieces are 16 bytes instead of 8 (641 rows, 64 fields, analysis /
  // synthesis: 3200 439 / 502 -> 356 / 405 us, 4000 587 / 609 -> 441 / 533)
  const bool two = value_size == 4 && lfc == 0 && vec && maxR > 3072 && maxF >= 2 && items_of(2) >= ncu &&
                   lds_of(2) <= kAnyMaxLds;
  if (two) lfc = 1;
  const int fc = 1 << lfc;
  return {lfc, two ? 1024 : holds(fc, 256) ? 256 : 512, vec, tw_of(fc), lds_of(fc)};
}

// Whether a length's group kernel (fc fields per item) takes a level rather
// than the any-length kernel, which has smaller items: not where the groups
// are mostly empty (2 fc > 3 F) and there is an item for every compute unit,
// so that the empty sequences cost time (1 field, 641 rows, analysis: I = 1920
// FP32 21.9 us, any-length 16.0; I = 1600 FP64 21.5, 16.4).  With fewer items
// than units they cost none, and the fixed radices win: I = 960 FP64, 479 rows,
// 3 fields 14 us (any-length 18); over 3942 plans of all lengths with 16..641
// rows and 1..20 fields the any-length kernels take 1.1 to 1.6 times as long
// per length.
inline bool group_takes(int fc, const LevelDesc& L, int ncu) {
  return 2 * fc <= 3 * L.F || (long long)L.Jh * ((L.F + fc - 1) / fc) < ncu;
}

// Whether the analysis of a level goes to the register-held kernels of
// sht_fft.hip (8 fields per item in FP32, 4 in FP64, lengths 2160..3072)
// rather than to the group kernel.  Those hold 4 (2) fields there and write
// the workspace in 32-byte pieces, which costs once it no longer fits the 256
// MB of memory-side cache; the held kernels write whole 64-byte runs, but have
// half the items, work through 8 (4) fields whether they exist or not, and
// spill in FP64 from 1024 wavenumbers on.  Both sides measured (us, group /
// held; ws = bytes of workspace):
//  FP32, from 120 MB where Cp is a multiple of 128, from 400 MB
//   elsewhere, and from 250 MB below 2560 in the first case only:
//   2880, 1919 rows, 64 fields 710 / 579, 32 fields 313 / 300; 3072, 2049
//   rows, 64 fields 847 / 634, 128 rows, 128 fields (134 MB) 119 / 109; 2880,
//   641 rows, 8 fields 37 / 52, 1 field half the time; 2304, 320 rows, 128
//   fields (252 MB) 200 / 185, N = 1151, 641 rows, 64 fields 240 / 208; 2160,
//   64 and 128 fields up to 240 MB 6-17 % longer; 2160..2400 with 96 fields
//   (Cp = 192) 3-12 % longer at any size.
//  FP64, where Cp is a multiple of 128 from 90 MB, else of 64 from
//   230 MB; at three wavenumbers per thread the former from 400 MB and not at
//   2160: 2880, 1919 rows, 64 fields 1473 / 1164, 32 fields 702 / 597; 2304,
//   128 rows, 64 fields 79 / 67; 2880, N = 1439, 641 rows, 64 fields 659 / 581,
//   32 fields 314 / 312; 2160, N = 1079, 641 rows, 128 fields 832 / 983; few
//   fields or rows (2880, 641 rows, 8 fields) 63 / 82.  3072, where the runs
//   spill at two wavenumbers too, gains nothing (1745 / 1697, else equal).
//  No synthesis: beside the group kernels that hold the reduced transform's
//   limits, 2880, FP64, N = 959, 1919 rows, 64 fields 1337 / 1350, N = 639
//   1124 / 1232, N = 300 809 / 910; only with up to 16 items of 4 fields per
//   unit and N >= 959 up to 5 % shorter (511 rows, 16 fields, N = 1023 96 /
//   92, N = 959 92.5 / 91.9).
inline bool held_takes(bool dbl, const LevelDesc& L) {
  const int I = L.I;
  if (I != 2160 && I != 2304 && I != 2400 && I != 2560 && I != 2880 && I != 3072) return false;
  const double ws = 2.0 * L.Jh * (L.N + 1) * L.Cp * (dbl ? 8 : 4);
  const bool c128 = L.Cp % 128 == 0;
  if (!dbl) return c128 ? ws >= (I >= 2560 ? 120e6 : 250e6) : I >= 2560 && ws >= 400e6;
  if (I == 3072) return false;
  if (L.N >= 1024) return c128 && I > 2160 && ws >= 400e6;
  return c128 ? ws >= 90e6 : L.Cp % 64 == 0 && ws >= 230e6;
}

// Whether a level of a multi-level plan shares the any-length launch with
// others like it: no group kernel, one that does not take it, or fewer items
// of it than compute units.
inline bool level_shares(bool dbl, bool analysis, const LevelDesc& L, int ncu) {
  const int fc = group_fields(dbl, analysis, L.I);
  return fc == 0 || !group_takes(fc, L, ncu) || (long long)L.Jh * ((L.F + fc - 1) / fc) < ncu;
}

// Whether a multi-level plan's zonal stage defaults to one launch over all
// levels (k_zonal_levels) where they allow it: in FP64 with 3 to 8 fields, at
// least 1.85 items of 4 fields per compute unit and a level that would share
// the any-length launch.  One launch / per length in us (cc_poles grids from I
// = 100 doubling): five levels, 3 fields, synthesis 45 / 58, 5 fields 73 / 83,
// 8 fields 80 / 89, analysis 37 / 52, 65 / 82, 71 / 92; four levels, 5 fields
// 30 / 33 and 27 / 34; three levels (0.9 to 1.8 items), 3 fields, synthesis 13
// / 11; 12 fields, synthesis 128 / 123; FP32 synthesis 1.0 to 2.3 times as
// long.
inline bool one_launch_default(bool dbl, bool analysis, int nlev, const LevelDesc* lev, int ncu) {
  if (!dbl) return false;
  double items = 0;
  bool fields = true, share = false;
  for (int l = 0; l < nlev; ++l) {
    items += (double)lev[l].Jh * ((lev[l].F + 3) / 4);
    fields = fields && lev[l].F >= 3 && lev[l].F <= 8;
    share = share || level_shares(dbl, analysis, lev[l], ncu);
  }
  return nlev > 1 && fields && share && items >= 1.85 * ncu;
}

}  // namespace sht

#endif  // SHT_ZONAL_RULE_H_
