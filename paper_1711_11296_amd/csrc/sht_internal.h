// Internal declarations shared by the host planner, the kernels and the C ABI.
#ifndef SHT_INTERNAL_H_
#define SHT_INTERNAL_H_

#include <cstddef>
#include <cstdint>
#include <cstring>
#include <type_traits>

#include "../../include/sht.h"

#define SHT_MAX_LEVELS 8
#define SHT_MAX_RADICES 6
#define SHT_MAX_I 4096

// Latitude (contraction) dimension of the table and workspace is padded to a
// multiple of this.
#define SHT_K_PAD 32

namespace sht {

// ---- host planning (sht_host.cpp) ----
bool grid_args_ok(int J, int kind);
void grid_nodes(int J, int kind, double* mu, double* sint);
void grid_weights(int J, int kind, double* w);
void alf_column(int N, int m, int nr, const double* mu, const double* sint,
                double* out, long ld);
void alf_table(int N, int nr, const double* mu, const double* sint,
               double* out, int nthreads);
bool factor_radices(int I, int* rad, int* nrad);

// ---- device-side descriptors ----

// One transform level as the kernels see it.
struct LevelDesc {
  int N, J, I, F;
  int Jh;      // ceil(J/2): folded rows (northern rows incl. equator)
  int Kp;      // Jh padded to SHT_K_PAD
  int Cp;      // workspace row length (columns = 2F padded)
  int nrad;
  int rad[SHT_MAX_RADICES];   // radix of each Stockham pass
  int pns[SHT_MAX_RADICES];   // product of the radices of the earlier passes
  int ptw[SHT_MAX_RADICES];   // twiddle index stride I / (pns * rad)
  unsigned pmag[SHT_MAX_RADICES];  // floor((2^32-1)/pns) + 1 (0 when pns == 1)
  int pnb[SHT_MAX_RADICES];        // butterflies per sequence, I / rad
  unsigned pbm[SHT_MAX_RADICES];   // floor((2^32-1)/pnb) + 1 (0 when pnb == 1)
  unsigned ivm;                    // the same for the vectors of a grid row (set at launch)
  int fft_item0;   // first FFT work item of this level
  int nfb;         // field blocks of the FFT kernels
  int m_base;      // index of (level, m=0) in the per-m offset arrays
  int zk;          // zonal stage, one-launch multi-level kernel: configuration of this level (set at launch)
  int wsh;         // log2 of the analysis workspace column block W = min(2 FB, 16) (ws_col)
  long long grid_off;  // element offset of this level in the grid buffer
  long long spec_off;  // element offset of this level in the spec buffer
  long long ws_off;    // element offset in the workspace
  long long wblk;      // workspace elements from one wavenumber's region to the next (ws_block)
  long long wjb;       // and from one block of 32 latitude rows to the next, (N + 1) wblk
  const void* tw;      // I twiddles exp(-2 pi i k / I), complex, data type
  const double* wrow;  // Jh quadrature weights of the northern rows
  const double* murow; // Kp nodes mu_j of the northern rows, zero past Jh (analysis with generated P~)
};

// Kernel arguments, for NL levels: a launch over one level passes one
// descriptor instead of eight (a launch with 2.7 KB of arguments takes the
// host 4.1 us, one with 512 bytes 3.1 us).
template <int NL>
struct FftArgsN {
  int nlev;
  int nitems;
  const void* src;   // grid (analysis) or workspace (synthesis)
  void* dst;         // workspace (analysis) or grid (synthesis)
  // scalars: value *= (use_w ? w_j : 1) * (use_inv_I ? 1/I : 1) * (m ? mscale : 1)
  int use_w;
  int use_inv_I;
  double mscale;
  int tw_lds;        // element offset of the LDS twiddle table (set at launch)
  int fb;            // fields per work item (zonal_fields_per_block)
  int lfc;           // any-length kernels: log2 of the fields per item (set at launch)
  int one_launch;    // multi-level plans: one launch over all levels where they allow it
  // per (level, m): first latitude of the Legendre sums (reduced transform;
  // null otherwise); the synthesis leaves whole 128-latitude tiles below it
  // out of the workspace, and the zonal synthesis reads them as zero
  const int* jstart;
  LevelDesc lev[NL];
};
typedef FftArgsN<SHT_MAX_LEVELS> FftArgs;
typedef FftArgsN<1> FftArgs1;


// One work tile of a Legendre kernel; level < 0 marks an idle slot.
struct Tile {
  int level, m, rb, cb;
};

template <int NL>
struct GemmArgsN {
  int nlev;
  int ntiles;
  const Tile* tiles;           // one per workgroup
  const long long* tab_off;    // per (level, m): element offset of the table block
  const void* table;           // P~ table copy (FP64 in the FP64 form, else FP32)
  const int* jstart;           // per (level, m): first latitude of the sums (reduced transform; else 0)
  const void* spec_in;         // synthesis: spectra
  void* spec_out;              // analysis: spectra
  void* ws;                    // workspace
  // analysis with P~ generated in the kernel (FP64): per (level, m) the two
  // seed rows P~_{m+16g}, P~_{m+16g+1} of every 16-degree group g, each Kp
  // long, and the recurrence coefficients (A_r, B_r) of the rows r = n - m,
  // P~_n = A_r mu P~_{n-1} - B_r P~_{n-2}
  const double* seeds;
  const long long* seed_off;
  const double* rec;
  const long long* rec_off;
  LevelDesc lev[NL];
};
typedef GemmArgsN<SHT_MAX_LEVELS> GemmArgs;


// The arguments of a single-level launch (level 0 of a).
inline FftArgs1 one_level(const FftArgs& a) {
  FftArgs1 o;
  std::memcpy(&o, &a, sizeof(o));  // the levels come last, level 0 first
  o.nlev = 1;
  return o;
}
inline GemmArgsN<1> one_level(const GemmArgs& a) {
  GemmArgsN<1> o;
  std::memcpy(&o, &a, sizeof(o));
  o.nlev = 1;
  return o;
}
static_assert(std::is_trivially_copyable<FftArgs>::value && offsetof(FftArgs, lev) == offsetof(FftArgs1, lev) &&
                  std::is_trivially_copyable<GemmArgs>::value && offsetof(GemmArgs, lev) == offsetof(GemmArgsN<1>, lev),
              "one layout up to the levels");

// ---- kernel launchers (sht_fft.hip, sht_legendre.hip) ----
// The stream argument is a hipStream_t.
// Fields per column block of the analysis workspace (and per item of the
// zonal kernels that hold their runs in registers).
inline int zonal_fields_per_block(int form) { return form == SHT_FORM_FP64 ? 4 : 8; }
// Workspace layout (per level).  The latitude rows j < Kp come in blocks of
// 32; block jb holds, for every wavenumber m, one region of 32 rows of 2 Cp
// elements, the regions of consecutive m next to each other: region (jb, m)
// starts at jb wjb + m wblk, wjb = (N + 1) wblk.  The rows j >= ceil(J/2) of
// the last block stay zero.  A row holds the columns c = 2 field + {re, im}
// < Cp of both parities p.  (With all rows of one m in one region, a zonal
// item, which touches one row of every m, met another page at every
// wavenumber: regions 3 MB apart at T479 with 400 fields.  Blocks of 32 rows
// bring them within a few KB, and a Legendre tile still reads whole K blocks
// as one run.)
// The two directions use a region differently (each writes and reads its own):
// * synthesis (and forward adjoint): two planes, row r of the block at r Cp,
//   column c, the odd parity's plane ws_odd elements after the even one's:
//   behind the block's existing rows, so that the planes never overlap the
//   rows the analysis keeps zero;
// * analysis (and inverse adjoint): row r at 2 r Cp holds both parities in
//   blocks of W = 2^wsh = min(2 FB, 16) columns, [column block][parity][W]
//   (ws_col): the stores of a block's FB fields for one m are one contiguous
//   run of 4 FB elements (128 bytes), and each latitude row of a Legendre
//   analysis tile is one run over both parities.
// Offset of (parity, column c) within an analysis row:
constexpr int ws_col(int wsh, int par, int c) {
  return ((c >> wsh) << (wsh + 1)) + (par << wsh) + (c & ((1 << wsh) - 1));
}
// A region's 32 rows plus a pad of 256 bytes: an odd number of 256-byte
// pieces, so that the regions of consecutive wavenumbers (one wave's lanes in
// the zonal kernels) start on different HBM channels.
constexpr long long ws_block(long long Cp, int elem, bool pad) {
  return 2LL * SHT_K_PAD * Cp + (pad ? 256 / elem : 0);
}
// Synthesis: offset of the odd-parity plane in a region of block jb; in a
// whole block half the region's pad lies between the planes (the two loads of
// one wavenumber would otherwise meet the same channel).
constexpr long long ws_odd(int Jh, long long Cp, long long wblk, int jb) {
  return Jh - SHT_K_PAD * jb < SHT_K_PAD ? (Jh - SHT_K_PAD * jb) * Cp : wblk / 2;
}
// The fixed-length zonal kernels address the workspace with 32-bit byte
// offsets from a per-wave base: 64 regions must stay below 4 GiB (else the
// any-length kernels run).
inline bool zonal_offsets_fit(long long wblk, long long elem) { return 64.0 * (double)wblk * (double)elem < 4294967296.0; }
// Lengths 16 R2 R3 of a single level (sht_group.h): -1 where these kernels do
// not take the level, else a hipError_t; ncu compute units.
int launch_zonal_group_analysis_f32(const FftArgs1& a, int ncu, void* stream);
int launch_zonal_group_synthesis_f32(const FftArgs1& a, int ncu, void* stream);
int launch_zonal_group_analysis_f64(const FftArgs1& a, int ncu, void* stream);
int launch_zonal_group_synthesis_f64(const FftArgs1& a, int ncu, void* stream);
// Any lengths (sht_zonal_any.hip); ncu compute units.
int launch_zonal_any(bool dbl, bool analysis, const FftArgs& a, int ncu, void* stream);
int launch_zonal(int form, bool analysis, const FftArgs& a, int maxN, void* stream);
// gen: generate P~ in the kernels from the plan's seed rows instead of
// reading a table (plan option otf)
int launch_legendre(int form, bool analysis, const GemmArgs& g, int ncb, bool gen, void* stream);
// Transfers between truncations and nested grids (sht_transfer.hip).
int launch_retruncate(int Nin, int Nout, int F, bool dbl, const void* in, void* out, void* stream);
int launch_inject(int Jf, int If, int Jc, int Ic, int F, int rs, int r0, int cs, bool dbl, const void* fine,
                  void* coarse, void* stream);
// Zero units [first16, first16 + len16) (16-byte units) of nplanes planes
// spaced pitch16 units apart, starting at base (16-byte aligned).
int launch_clear_span(void* base, long long nplanes, long long pitch16, long long first16, long long len16,
                      void* stream);
int launch_product(long long n, bool dbl, const void* a, const void* b, void* out, void* stream);
int launch_laplacian(int N, int F, double scale, bool dbl, const void* in, void* out, void* stream);
int launch_residual(long long n, long long n_per, double alpha, bool dbl, const void* x, const void* kappa,
                    const void* y, const void* f, void* r, void* stream);
// Widest column blocking (16-column units) a Legendre kernel of a form takes
// (wider tiles do not fit the register file).
inline int max_ncb(int form, bool analysis) { return form == SHT_FORM_FP32 && analysis ? 10 : 8; }

}  // namespace sht

#endif  // SHT_INTERNAL_H_
