// Zonal (longitude) stage of the transform pair, with the equatorial parity
// fold of App. B fused in.
//
// Analysis, Sec. 2 (discretised zonal integral, 1/I convention): for the
// mirror pair of rows (j, J-1-j) the kernel forms z = x_north + i x_south,
// runs one complex FFT of length I in LDS (Stockham), and
// separates the two real spectra:
//   X_north^m = (Z^m + conj Z^{I-m}) / 2,  X_south^m = (Z^m - conj Z^{I-m}) / 2i.
// It then writes the symmetric and antisymmetric parts of App. B (eqs. B3,
// B4), already multiplied by the quadrature weight:
//   S^m_j = w_j (X_north^m + X_south^m),  A^m_j = w_j (X_north^m - X_south^m);
// the equator row (odd J) gives S = w X_eq and A = 0.
//
// Synthesis: the reverse.  From S and A (the Legendre sums of Sec. 2,
// eq. iLT, split by parity) the kernel rebuilds X_north = S + A and
// X_south = S - A, packs Z^m = X_north^m + i X_south^m and its Hermitian
// partner at I-m, and one inverse FFT yields both rows:
//   x(lambda_i) = Re X^0 + 2 sum_{m>=1} Re(X^m e^{i m lambda_i}).
//
// Three families of kernels: sht_group.h (lengths 16 R2 R3 known at compile
// time), sht_any.h (any length), and here the analysis kernels that hold their
// runs in registers, which some lengths past 2048 use (launch_held), with the
// choice of kernel and the multi-level launches.
//
// Work decomposition of the kernels here: one workgroup per (mirror row
// pair, block of FB fields).  The FB fields go through the LDS buffer one after the other and
// the wavenumbers m <= N of all FB fields are kept in registers, so that each
// workspace access is a contiguous run of 2*FB values (64 bytes) per (m,
// parity, row) instead of one isolated complex value; the analysis stores
// both parities of a row as one run of 4*FB values (ws_col).
//
// Workspace layout (per level): see ws_col and ws_block; the analysis and
// the synthesis lay it out differently.

#include <hip/hip_runtime.h>

#include <type_traits>
#include <utility>

#include "sht_internal.h"
#include "sht_any.h"
#include "sht_dft.h"
#include "sht_group.h"

namespace sht {

// The workspace run of one (wavenumber, parity, latitude pair, field block)
// is 2 FB values = 64 bytes, and the thread of wavenumber m holds the whole
// run; consecutive lanes hold consecutive m, whose runs are a plane apart.
// Before storing, the four lanes of each quad exchange 16-byte pieces so
// that lane j holds piece j of the four runs of its quad; a 16-byte store
// instruction then covers 16 whole runs instead of touching 64 cache lines.
constexpr int kQuadXor1 = 0xB1;  // DPP quad_perm [1,0,3,2]
constexpr int kQuadXor2 = 0x4E;  // DPP quad_perm [2,3,0,1]

// 4x4 transpose of 16-byte pieces across a quad; its own inverse.  Every
// lane of the quad must take part.
__device__ __forceinline__ void quad_transpose(int (&x)[4][4]) {
  const int j = threadIdx.x & 3;
  const bool h1 = (j & 1) != 0, h2 = (j & 2) != 0;
#pragma unroll
  for (int p = 0; p < 4; p += 2)
#pragma unroll
    for (int d = 0; d < 4; ++d) {
      const int v = h1 ? x[p][d] : x[p + 1][d];
      const int r = __builtin_amdgcn_update_dpp(0, v, kQuadXor1, 0xF, 0xF, false);
      if (h1)
        x[p][d] = r;
      else
        x[p + 1][d] = r;
    }
#pragma unroll
  for (int p = 0; p < 2; ++p)
#pragma unroll
    for (int d = 0; d < 4; ++d) {
      const int v = h2 ? x[p][d] : x[p + 2][d];
      const int r = __builtin_amdgcn_update_dpp(0, v, kQuadXor2, 0xF, 0xF, false);
      if (h2)
        x[p][d] = r;
      else
        x[p + 2][d] = r;
    }
}

// Store the runs v of the quad's four wavenumbers m - j .. m - j + 3
// (j = lane in quad) at dst(m') = base + m' * region; runs with m' > N
// are skipped.  All lanes of the quad must call it.  base is uniform and the
// 64 lanes of a wave hold consecutive wavenumbers: each address is a
// uniform 64-bit base at the wave's first wavenumber plus a 32-bit per-lane
// byte offset of fewer than 64 regions (zonal_offsets_fit).
template <typename T, int FB>
__device__ __forceinline__ void store_runs_quad(T* base, long long region, int m, int N,
                                                const cx<T> (&v)[FB]) {
  static_assert(2 * FB * (int)sizeof(T) == 64, "64-byte runs");
  const int lane = threadIdx.x & 63, j = lane & 3;
  const long long step64 = region * (long long)sizeof(T);
  const int mw = __builtin_amdgcn_readfirstlane(m - lane);  // the wave's first wavenumber
  char* b = reinterpret_cast<char*>(base) + (long long)mw * step64;
  const unsigned step = (unsigned)step64;
  int x[4][4];
  __builtin_memcpy(x, v, 64);
  quad_transpose(x);
  unsigned off = (unsigned)(lane - j) * step + 16u * (unsigned)j;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int mr = m - j + r;
    if (mr <= N) {
      typedef int i32x4 __attribute__((ext_vector_type(4)));
      *reinterpret_cast<i32x4*>(b + off) = i32x4{x[r][0], x[r][1], x[r][2], x[r][3]};
    }
    off += step;
  }
}

// ---------------------------------------------------------------------------
// Fixed-length transforms: I = 16 R2 R3 in three passes with compile-time
// radices, twiddle strides and index arithmetic (Plan3; the passes are those
// of sht_group.h with a field stride of IP).  The grid rows are loaded
// straight into the registers of the first pass.
// ---------------------------------------------------------------------------
template <typename T, class P, int NT, int FC>
struct Fft3 {
  static constexpr int S1 = (FC * P::nb1 + NT - 1) / NT;
  static constexpr int S2 = (FC * P::nb2 + NT - 1) / NT;
  static constexpr int S3 = (FC * P::nb3 + NT - 1) / NT;

  // twiddles of passes two and three from the table exp(-2 pi i e / I)
  static __device__ void stage_twiddles(cx<T>* twl, const cx<T>* __restrict__ twg) {
    for (int x = threadIdx.x; x < P::ntw; x += NT) {
      int e;
      if (x < P::tw3) {
        const int t = x / P::Ns2 + 1, k = x - (t - 1) * P::Ns2;
        e = t * k * P::R3;
      } else {
        const int y = x - P::tw3;
        const int t = y / P::Ns3 + 1, k = y - (t - 1) * P::Ns3;
        e = t * k;
      }
      twl[x] = twg[e];
    }
  }

  // first pass on values already in registers (v[s] = inputs j + t nb1 of
  // slot s); results stored in the padded order
  static __device__ __forceinline__ void pass1_store(cx<T> (&v)[S1][16], cx<T>* buf) {
#pragma unroll
    for (int s = 0; s < S1; ++s) {
      const int u = threadIdx.x + s * NT;
      if (u < FC * P::nb1) {
        const int f = u / P::nb1, j = u - f * P::nb1;
        Dft<T, 16>::run(v[s]);
        cx<T>* d = buf + f * P::IP + 17 * j;
#pragma unroll
        for (int t = 0; t < 16; ++t) d[t] = v[s][t];
      }
    }
  }

  // second pass: padded order in, natural order out (in place)
  static __device__ __forceinline__ void pass2(cx<T>* buf, const cx<T>* twl) {
    constexpr int R = P::R2;
    cx<T> v[S2][R];
#pragma unroll
    for (int s = 0; s < S2; ++s) {
      const int u = threadIdx.x + s * NT;
      if (u < FC * P::nb2) {
        const int f = u / P::nb2, j = u - f * P::nb2;
        const cx<T>* src = buf + f * P::IP + j + (j >> 4);
#pragma unroll
        for (int t = 0; t < R; ++t) v[s][t] = src[t * P::S2P];
        const cx<T>* w = twl + P::tw2 + (j & 15);
#pragma unroll
        for (int t = 1; t < R; ++t) v[s][t] = cmul(v[s][t], w[(t - 1) * P::Ns2]);
        Dft<T, R>::run(v[s]);
      }
    }
    __syncthreads();
#pragma unroll
    for (int s = 0; s < S2; ++s) {
      const int u = threadIdx.x + s * NT;
      if (u < FC * P::nb2) {
        const int f = u / P::nb2, j = u - f * P::nb2;
        cx<T>* d = buf + f * P::IP + (j >> 4) * (16 * R) + (j & 15);
#pragma unroll
        for (int t = 0; t < R; ++t) d[t * 16] = v[s][t];
      }
    }
    __syncthreads();
  }

  // third pass into registers: v[s][t] is element j + t Ns3 of field f,
  // (f, j) = slot s of this thread
  static __device__ __forceinline__ void pass3_regs(cx<T> (&v)[S3][P::R3], const cx<T>* buf,
                                                    const cx<T>* twl) {
    constexpr int R = P::R3;
#pragma unroll
    for (int s = 0; s < S3; ++s) {
      const int u = threadIdx.x + s * NT;
      if (u < FC * P::nb3) {
        const int f = u / P::nb3, j = u - f * P::nb3;
        const cx<T>* src = buf + f * P::IP + j;
#pragma unroll
        for (int t = 0; t < R; ++t) v[s][t] = src[t * P::nb3];
        const cx<T>* w = twl + P::tw3 + j;
#pragma unroll
        for (int t = 1; t < R; ++t) v[s][t] = cmul(v[s][t], w[(t - 1) * P::Ns3]);
        Dft<T, R>::run(v[s]);
      }
    }
  }
};

// The slots item, item + G, ... of the level.
template <typename T, class P, int NT, int FB, int FC, int MS>
__device__ __forceinline__ void zonal_analysis_run_p3(const FftArgs1& a, int item, unsigned char* smem_raw) {
  using F3 = Fft3<T, P, NT, FC>;
  constexpr int NRD = FB / FC, I = P::I;
  cx<T>* buf = reinterpret_cast<cx<T>*>(smem_raw);
  cx<T>* twl = buf + FC * P::IP;
  const LevelDesc& L = a.lev[0];
  const int s0 = 0, end = a.nitems, n = end;
  const T* grid = static_cast<const T*>(a.src) + L.grid_off;
  T* ws = static_cast<T*>(a.dst) + L.ws_off;
  const T msc = (T)a.mscale;
  const int N = L.N, J = L.J;

  if (item >= end) return;
  F3::stage_twiddles(twl, static_cast<const cx<T>*>(L.tw));

  cx<T> v1[F3::S1][16];
  auto load_rows = [&](int slot, int rd) __attribute__((always_inline)) {
    const int itm = xcd_map(slot - s0, n);
    const int jp = itm / L.nfb, fb = itm - jp * L.nfb;
    const bool eq = (J & 1) && (jp == (J >> 1));
#pragma unroll
    for (int s = 0; s < F3::S1; ++s) {
      const int u = threadIdx.x + s * NT;
      if (u < FC * P::nb1) {
        const int f = u / P::nb1, j = u - f * P::nb1;
        const int fld = fb * FB + rd * FC + f;
        const bool valid = fld < L.F;
        const T* rn = grid + ((long long)fld * J + jp) * I + j;
        const T* rs = grid + ((long long)fld * J + (J - 1 - jp)) * I + j;
#pragma unroll
        for (int t = 0; t < 16; ++t) {
          v1[s][t].x = valid ? rn[t * P::nb1] : (T)0;
          v1[s][t].y = (valid && !eq) ? rs[t * P::nb1] : (T)0;
        }
      }
    }
  };

  load_rows(item, 0);
  for (; item < end; item += gridDim.x) {
    const int itm = xcd_map(item - s0, n);
    const int jp = itm / L.nfb, fb = itm - jp * L.nfb;
    const bool eq = (J & 1) && (jp == (J >> 1));
    const T rscale = row_scale<T>(a, L, jp);
    const int next = item + (int)gridDim.x;

    cx<T> stS[MS][FB], stA[MS][FB];
#pragma unroll
    for (int rd = 0; rd < NRD; ++rd) {
      F3::pass1_store(v1, buf);
      __syncthreads();
      if (rd + 1 < NRD)
        load_rows(item, rd + 1);
      else if (next < end)
        load_rows(next, 0);
      F3::pass2(buf, twl);
      {
        cx<T> v3[F3::S3][P::R3];
        F3::pass3_regs(v3, buf, twl);
        __syncthreads();
        // only the bins m <= N and I - m (m <= N) are used by the fold
#pragma unroll
        for (int s = 0; s < F3::S3; ++s) {
          const int u = threadIdx.x + s * NT;
          if (u < FC * P::nb3) {
            const int f = u / P::nb3, j = u - f * P::nb3;
            cx<T>* d = buf + f * P::IP + j;
#pragma unroll
            for (int t = 0; t < P::R3; ++t) {
              const int pos = j + t * P::Ns3;
              if (pos <= N || pos >= I - N) d[t * P::Ns3] = v3[s][t];
            }
          }
        }
        __syncthreads();
      }
#pragma unroll
      for (int s = 0; s < MS; ++s) {
        const int m = threadIdx.x + s * NT;
#pragma unroll
        for (int fc = 0; fc < FC; ++fc) {
          cx<T> S = {(T)0, (T)0}, A = {(T)0, (T)0};
          if (m <= N) {
            const cx<T> Pm = buf[fc * P::IP + m];
            cx<T> Q = buf[fc * P::IP + (m == 0 ? 0 : I - m)];
            Q.y = -Q.y;  // conj Z^{I-m}
            const T h = (T)0.5;
            const cx<T> Xn = {h * (Pm.x + Q.x), h * (Pm.y + Q.y)};
            const cx<T> Xs = {h * (Pm.y - Q.y), -h * (Pm.x - Q.x)};
            const T sc = m == 0 ? rscale : rscale * msc;
            S = cx<T>{sc * (Xn.x + Xs.x), sc * (Xn.y + Xs.y)};
            A = cx<T>{sc * (Xn.x - Xs.x), sc * (Xn.y - Xs.y)};
            if (m == 0) {
              S.y = (T)0;
              A.y = (T)0;
            }
            if (eq) A = cx<T>{(T)0, (T)0};
          }
          stS[s][rd * FC + fc] = S;
          stA[s][rd * FC + fc] = A;
        }
      }
      __syncthreads();
    }

    const long long Cp = L.Cp;
    const long long plane = L.wblk;
    // the item's column block (ws_col): even run, then odd run
    T* wrow = ws + (jp / SHT_K_PAD) * L.wjb + (long long)(jp % SHT_K_PAD) * 2 * Cp + 4 * fb * FB;
#pragma unroll
    for (int s = 0; s < MS; ++s) {
      const int m = threadIdx.x + s * NT;
      store_runs_quad<T, FB>(wrow, plane, m, N, stS[s]);
      store_runs_quad<T, FB>(wrow + 2 * FB, plane, m, N, stA[s]);
    }
  }
}

template <typename T, class P, int NT, int FB, int FC, int MS>
__global__ __launch_bounds__(NT) void k_zonal_analysis_p3(const FftArgs1 a) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  zonal_analysis_run_p3<T, P, NT, FB, FC, MS>(a, blockIdx.x, smem_raw);
}

// ---------------------------------------------------------------------------
// Multi-level plans in one launch.  A configuration says how a level runs:
// with a compile-time three-pass plan (ZGrp) or with runtime radices (ZRt).
// The persistent workgroups of k_zonal_levels walk their slots in increasing
// order, which visits the levels one after the other, each as a contiguous
// run of slots (every level's items are spread over all XCDs, see xcd_map);
// a run is handed to the level's configuration (LevelDesc::zk), and the LDS
// is reused by the next run after a barrier.  One launch therefore covers
// every level, with no idle tail between levels.
// ---------------------------------------------------------------------------
template <class P, int FC>
struct ZGrp {
  static constexpr int fc = FC;
  template <typename T, int NT>
  static constexpr size_t lds() {
    return Grp<T, P, NT, FC, false>::lds();
  }
  template <typename T, int NT, int FB, bool ANA>
  static __device__ __forceinline__ int run(const FftArgs& a, int l, int item, unsigned char* smem) {
    if constexpr (ANA)
      return Grp<T, P, NT, FC, false>::analysis(a, l, item, smem);
    else
      return Grp<T, P, NT, FC, false>::synthesis(a, l, item, smem);
  }
};

// runtime radices (sht_any.h)
template <bool VEC, int MAXI>
struct ZRt {
  static constexpr int maxi = MAXI;
  template <typename T, int NT, int FB, bool ANA>
  static __device__ __forceinline__ int run(const FftArgs& a, int l, int item, unsigned char* smem) {
    constexpr int VW = sizeof(T) == 4 ? 2 : 1;
    if constexpr (ANA)
      return any_analysis_run<T, NT, VEC, VW>(a, item, level_end(a, l), smem);
    else
      return any_synthesis_run<T, NT, VEC, VW>(a, item, level_end(a, l), smem);
  }
};

template <typename T, int NT, int FB, bool ANA, class C, class... Cs>
__device__ __forceinline__ int zonal_run_cfg(const FftArgs& a, int k, int l, int item, unsigned char* smem) {
  if (k == 0) return C::template run<T, NT, FB, ANA>(a, l, item, smem);
  if constexpr (sizeof...(Cs) > 0)
    return zonal_run_cfg<T, NT, FB, ANA, Cs...>(a, k - 1, l, item, smem);
  else
    return level_end(a, l);  // (not reached: the launcher gives every level a configuration)
}

template <typename T, int NT, int FB, bool ANA, class... Cs>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 4 ? 4 : 2))) void k_zonal_levels(const FftArgs a) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  int item = blockIdx.x;
  while (item < a.nitems) {
    const int l = level_of(a, item);
    item = zonal_run_cfg<T, NT, FB, ANA, Cs...>(a, a.lev[l].zk, l, item, smem_raw);
    __syncthreads();  // the next level's run refills the LDS
  }
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
// LDS per workgroup on gfx950 is 160 KiB; above 64 KiB a kernel has to opt in.
constexpr size_t kMaxLds = 160 * 1024;

template <auto Kernel>
static void lds_optin(size_t bytes) {
  static size_t done = 0;  // one flag per kernel instantiation
  if (bytes > 65536 && bytes > done) {
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(Kernel),
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
    done = bytes;
  }
}

static int g_num_cu = 0;

template <typename T, class P, int NT, int FB, int FC, int MS>
static hipError_t launch_p3_ms(const FftArgs1& a, hipStream_t st) {
  const size_t lds = (size_t)(FC * P::IP + P::ntw) * sizeof(cx<T>);
  int per_cu = (int)(kMaxLds / lds);
  const int by_waves = 2048 / NT;
  per_cu = per_cu < by_waves ? per_cu : by_waves;
  per_cu = per_cu < 1 ? 1 : per_cu;
  int nwg = g_num_cu * per_cu;
  nwg = nwg < a.nitems ? nwg : a.nitems;
  const dim3 grid(nwg), block(NT);
  lds_optin<k_zonal_analysis_p3<T, P, NT, FB, FC, MS>>(lds);
  hipLaunchKernelGGL((k_zonal_analysis_p3<T, P, NT, FB, FC, MS>), grid, block, lds, st, a);
  return hipGetLastError();
}

// Two fields per round (four spill registers and cost ~5 %) on 512 threads.
template <typename T, int FB, class P>
static hipError_t launch_p3(const FftArgs1& a, int maxN, hipStream_t st) {
  constexpr int NT = 512, FC = 2;
  constexpr int MSMAX = ((P::I + 1) / 2 + NT - 1) / NT;  // N + 1 <= (I + 1) / 2
  static_assert(MSMAX == 3, "wavenumbers per thread");
  const int nm = maxN + 1;
  if (nm > 2 * NT) {
    if constexpr (sizeof(T) == 8 && P::I == 2160) return hipErrorInvalidValue;  // (held_takes: not taken)
    else return launch_p3_ms<T, P, NT, FB, FC, 3>(a, st);
  }
  if (nm > NT) return launch_p3_ms<T, P, NT, FB, FC, 2>(a, st);
  return launch_p3_ms<T, P, NT, FB, FC, 1>(a, st);
}

// The levels that held_takes gives to the register-held kernels.  FP64
// analysis takes the larger radix second: beside the runs a thread then holds
// 12 values of the last pass, not 15 (2880, 64 fields, 1919 rows: 1567 us with
// radix 15 last, 102 spills; 1172 with 6).  Spills at two / three wavenumbers
// per thread: FP64 analysis 0..10 / 13..48 registers, the others none.
template <typename T, int FB>
static bool launch_held(const FftArgs1& a, int maxN, hipStream_t st, hipError_t* err) {
  if (!held_takes(sizeof(T) == 8, a.lev[0])) return false;
  constexpr bool dbl = sizeof(T) == 8;
  switch (a.lev[0].I) {
    case 2160: *err = launch_p3<T, FB, Plan3<2160, dbl ? 15 : 9, dbl ? 9 : 15>>(a, maxN, st); return true;
    case 2304: *err = launch_p3<T, FB, Plan3<2304, 12, 12>>(a, maxN, st); return true;
    case 2400: *err = launch_p3<T, FB, Plan3<2400, dbl ? 15 : 10, dbl ? 10 : 15>>(a, maxN, st); return true;
    case 2560: *err = launch_p3<T, FB, Plan3<2560, 16, 10>>(a, maxN, st); return true;
    case 2880: *err = launch_p3<T, FB, Plan3<2880, dbl ? 15 : 12, dbl ? 12 : 15>>(a, maxN, st); return true;
    case 3072:
      if constexpr (!dbl) {
        *err = launch_p3<T, FB, Plan3<3072, 16, 12>>(a, maxN, st);
        return true;
      }
  }
  return false;
}

// Single-level plans whose I has a compile-time three-pass plan.
template <typename T, int FB>
static bool launch_fixed(bool analysis, const FftArgs& a, int maxN, hipStream_t st, hipError_t* err) {
  if (a.nlev != 1) return false;
  // the fixed-length kernels address the workspace with 32-bit offsets
  // from a per-wave base
  if (!zonal_offsets_fit(a.lev[0].wblk, sizeof(T))) return false;
  const FftArgs1 o = one_level(a);
  if (analysis && launch_held<T, FB>(o, maxN, st, err)) return true;
  const int e = sizeof(T) == 8 ? (analysis ? launch_zonal_group_analysis_f64(o, g_num_cu, st)
                                           : launch_zonal_group_synthesis_f64(o, g_num_cu, st))
                               : (analysis ? launch_zonal_group_analysis_f32(o, g_num_cu, st)
                                           : launch_zonal_group_synthesis_f32(o, g_num_cu, st));
  if (e < 0) return false;
  *err = (hipError_t)e;
  return true;
}

// compute units of the current device (persistent grids are sized by it)
static void ensure_num_cu() {
  if (g_num_cu == 0) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&g_num_cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        g_num_cu <= 0)
      g_num_cu = 256;
  }
}

template <typename T>
static hipError_t launch_generic(bool analysis, const FftArgs& a, hipStream_t st) {
  return (hipError_t)launch_zonal_any(sizeof(T) == 8, analysis, a, g_num_cu, st);
}

// The configurations of the one-launch kernel for one element type (zk =
// index into C1600, C800, C400, CRt) and its two instantiations.
template <typename T>
struct ZLevels {
  static constexpr bool dbl = sizeof(T) == 8;
  static constexpr int NT = 512;
  template <int I, int FC>
  using Z = ZGrp<Plan3<I, grp_r2(I, NT, FC), I / 16 / grp_r2(I, NT, FC)>, FC>;
  using C1600 = Z<1600, 4>;
  using C800 = Z<800, dbl ? 4 : 8>;
  using C400 = Z<400, dbl ? 4 : 8>;
  template <bool VEC>
  using CRt = ZRt<VEC, 1024>;
  template <int FB, bool ANA, bool VEC>
  static constexpr auto kernel() {
    return &k_zonal_levels<T, NT, FB, ANA, C1600, C800, C400, CRt<VEC>>;
  }
};

// Multi-level plans whose levels all have I = 1600, 800 or 400 (three-pass
// plans) or I <= 1024 (runtime radices), and at least two launches' worth of
// lengths: one launch of k_zonal_levels.  Returns false (nothing launched)
// for other plans.
template <typename T, int FB>
static bool launch_levels_one(bool analysis, const FftArgs& a, hipStream_t st, hipError_t* err) {
  constexpr int NT = ZLevels<T>::NT;
  using C1600 = typename ZLevels<T>::C1600;
  using C800 = typename ZLevels<T>::C800;
  using C400 = typename ZLevels<T>::C400;
  if (a.nlev < 2 || a.fb != FB) return false;
  FftArgs b = a;
  size_t lds = 0;
  int maxIrt = 0, maxNrt = 0, maxIP = 0, kinds = 0;
  bool vec = true;
  for (int l = 0; l < a.nlev; ++l) {
    const LevelDesc& L = a.lev[l];
    int k;
    size_t need = 0;
    if (L.I == 1600 || L.I == 800 || L.I == 400) {
      // the three-pass kernels address the workspace with 32-bit offsets
      // from a per-wave base
      if (!zonal_offsets_fit(L.wblk, sizeof(T))) return false;
      k = L.I == 1600 ? 0 : L.I == 800 ? 1 : 2;
      need = k == 0 ? C1600::template lds<T, NT>() : k == 1 ? C800::template lds<T, NT>() : C400::template lds<T, NT>();
      const int fc = k == 0 ? C1600::fc : k == 1 ? C800::fc : C400::fc;
      if ((double)fc * L.J * L.I * sizeof(T) >= 4294967296.0) return false;
      b.lev[l].nfb = (L.F + fc - 1) / fc;
    } else {
      if (L.I > ZLevels<T>::template CRt<true>::maxi || L.N + 1 > NT) return false;
      k = 3;
      const int r = any_nvec<16 / (int)sizeof(T)>(L.I) * (16 / (int)sizeof(T));
      maxIrt = r > maxIrt ? r : maxIrt;
      maxNrt = L.N > maxNrt ? L.N : maxNrt;
      const int ip = any_stride(L), V = 16 / (int)sizeof(T);
      maxIP = ip > maxIP ? ip : maxIP;
      vec = vec && L.I >= V;
    }
    kinds |= 1 << k;
    b.lev[l].zk = k;
    lds = need > lds ? need : lds;
  }
  // one runtime-radix launch or one length alone gains nothing
  if (__builtin_popcount(kinds) < 2) return false;
  if (maxIrt) {
    // a whole block of FB fields per item where it fits the kernels'
    // capacity per thread (AnyCap), else half of it
    constexpr int E = AnyCap<T>::E;
    b.lfc = FB == 8 ? 3 : 2;
    while ((maxIrt << b.lfc) > NT * E || (2 * (maxNrt + 1) << b.lfc) > NT * E) --b.lfc;
    b.tw_lds = ((maxIP << b.lfc) + 1) & ~1;
    const size_t rt = (size_t)(b.tw_lds + maxIrt) * sizeof(cx<T>);
    lds = rt > lds ? rt : lds;
  }
  long long items = 0;
  for (int l = 0; l < a.nlev; ++l) {
    LevelDesc& L = b.lev[l];
    if (L.zk == 3) {
      const int nv = vec ? any_nvec<16 / (int)sizeof(T)>(L.I) : L.I;
      L.ivm = nv > 1 ? 0xFFFFFFFFu / (unsigned)nv + 1u : 0u;
      L.nfb = (L.F + (1 << b.lfc) - 1) >> b.lfc;
    }
    L.fft_item0 = (int)items;
    items += (long long)L.Jh * L.nfb;
    if (items > 0x7fffffff) return false;
  }
  b.nitems = (int)items;
  int per_cu = (int)(kMaxLds / lds);
  constexpr int by_waves = (sizeof(T) == 4 ? 1024 : 512) / NT;  // waves per SIMD of k_zonal_levels
  per_cu = per_cu < by_waves ? per_cu : by_waves;
  per_cu = per_cu < 1 ? 1 : per_cu;
  int nwg = g_num_cu * per_cu;
  nwg = nwg < b.nitems ? nwg : b.nitems;
  const dim3 grid(nwg), block(NT);
  auto go = [&](auto ana, auto v) {
    constexpr auto K = ZLevels<T>::template kernel<FB, decltype(ana)::value, decltype(v)::value>();
    lds_optin<K>(lds);
    hipLaunchKernelGGL(K, grid, block, lds, st, b);
  };
  if (analysis)
    vec ? go(std::true_type{}, std::true_type{}) : go(std::true_type{}, std::false_type{});
  else
    vec ? go(std::false_type{}, std::true_type{}) : go(std::false_type{}, std::false_type{});
  *err = hipGetLastError();
  return true;
}

// Multi-level plans: one launch of k_zonal_levels where every level fits
// it (and FftArgs::one_launch asks for it); otherwise each level whose I has
// a compile-time three-pass plan gets a launch of its own (one level per
// argument block, its items renumbered from 0), and the other levels share
// one launch of the any-length kernel.  Levels with fewer items than compute
// units share that launch too, if there are two or more of them: side by side
// they cost less than one after the other on the faster kernels (FP32, 3
// fields, I = 400 and 200: 10.7 us, in two launches 15.4).  All launches go to
// the same stream, and the levels write disjoint parts of the output.
template <typename T, int FB>
static hipError_t launch_levels(bool analysis, const FftArgs& a, hipStream_t st) {
  hipError_t e1 = hipSuccess;
  if (a.one_launch && launch_levels_one<T, FB>(analysis, a, st, &e1)) return e1;
  auto single = [&](int l) {
    FftArgs one = a;
    one.nlev = 1;
    one.lev[0] = a.lev[l];
    one.lev[0].fft_item0 = 0;
    one.nitems = a.lev[l].Jh * a.lev[l].nfb;
    return one;
  };
  bool shared[SHT_MAX_LEVELS];
  int nshared = 0;
  for (int l = 0; l < a.nlev; ++l) nshared += shared[l] = level_shares(sizeof(T) == 8, analysis, a.lev[l], g_num_cu);
  FftArgs rest = a;
  rest.nlev = 0;
  rest.nitems = 0;
  for (int l = 0; l < a.nlev; ++l) {
    const FftArgs one = single(l);
    hipError_t e = hipSuccess;
    if ((!shared[l] || nshared == 1) && launch_fixed<T, FB>(analysis, one, a.lev[l].N, st, &e)) {
      if (e != hipSuccess) return e;
      continue;
    }
    rest.lev[rest.nlev] = a.lev[l];
    rest.lev[rest.nlev].fft_item0 = rest.nitems;
    rest.nitems += one.nitems;
    rest.nlev += 1;
  }
  if (rest.nlev == 0) return hipSuccess;
  return launch_generic<T>(analysis, rest, st);
}

template <typename T, int FB>
static hipError_t launch_zonal_t(bool analysis, const FftArgs& a, int maxN, hipStream_t st) {
  ensure_num_cu();
  if (a.nlev > 1) return launch_levels<T, FB>(analysis, a, st);
  hipError_t err = hipSuccess;
  if (launch_fixed<T, FB>(analysis, a, maxN, st, &err)) return err;
  return launch_generic<T>(analysis, a, st);
}

int launch_zonal(int form, bool analysis, const FftArgs& a, int maxN, void* stream) {
  hipStream_t st = static_cast<hipStream_t>(stream);
  // the kernels' item width must match every level's analysis column block
  const int fb = form == SHT_FORM_FP64 ? 4 : 8;
  for (int l = 0; l < a.nlev; ++l)
    if ((1 << a.lev[l].wsh) != (2 * fb < 16 ? 2 * fb : 16)) return (int)hipErrorInvalidValue;
  if (form == SHT_FORM_FP64) return (int)launch_zonal_t<double, 4>(analysis, a, maxN, st);
  return (int)launch_zonal_t<float, 8>(analysis, a, maxN, st);
}

}  // namespace sht
