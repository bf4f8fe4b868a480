// Zonal kernels of the lengths I = 16 R2 R3 (R2, R3 <= 16): the group scheme
// of sht_any.h with everything known at compile time.
//
// Work item = (mirror row pair, group of FC fields) on NT threads.  Analysis
// loads the rows straight into the registers of the radix-16 first pass
// (thread of butterfly j takes elements j + t I/16 of both rows, coalesced
// across the lanes) and folds from LDS to the workspace; synthesis unfolds
// the workspace into LDS and stores the last pass straight to the rows.
// Addresses are a uniform base plus a 32-bit lane offset.
//
// Bound: HBM, with the workspace's pieces scattered over the wavenumbers.
// Against the kernels that hold the S and A runs of 8 (16) fields in
// registers (sht_fft.hip; one 512-thread workgroup per compute unit at 190
// to 250 registers) nothing but the current pass lives in registers, so two
// or more workgroups, or one of 1024 threads, overlap their memory and
// compute phases.  GroupShape has the shapes and what they measured.
#ifndef SHT_GROUP_H_
#define SHT_GROUP_H_

#include <hip/hip_runtime.h>

#include "sht_any.h"
#include "sht_dft.h"
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

// field stride in LDS
template <class P>
constexpr int grp_stride() {
  return ((P::IP + 15) & ~15) + 2;
}

template <typename T, class P, int NT, int FC, bool PF>
struct Grp {
  static constexpr int I = P::I, GP = grp_stride<P>();
  static constexpr int VW = sizeof(T) == 4 && FC >= 2 ? 2 : 1, LV = FC / VW;
  static constexpr int S1 = (FC * P::nb1 + NT - 1) / NT, S2 = (FC * P::nb2 + NT - 1) / NT,
                       S3 = (FC * P::nb3 + NT - 1) / NT;
  static constexpr int UM = ((I + 1) / 2 * LV + NT - 1) / NT;
  static constexpr size_t lds() { return (size_t)(FC * GP + P::ntw) * sizeof(cx<T>); }

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
  static __device__ __forceinline__ void pass1_store(cx<T> (&v)[S1][16], cx<T>* buf) {
#pragma unroll
    for (int s = 0; s < S1; ++s) {
      const int u = (int)threadIdx.x + s * NT;
      if (u < FC * P::nb1) {
        const int f = u / P::nb1, j = u - f * P::nb1;
        Dft<T, 16>::run(v[s]);
        cx<T>* d = buf + f * GP + 17 * j;
#pragma unroll
        for (int t = 0; t < 16; ++t) d[t] = v[s][t];
      }
    }
  }
  static __device__ __forceinline__ void pass1_lds(cx<T>* buf) {
    cx<T> v[S1][16];
#pragma unroll
    for (int s = 0; s < S1; ++s) {
      const int u = (int)threadIdx.x + s * NT;
      if (u < FC * P::nb1) {
        const int f = u / P::nb1, j = u - f * P::nb1;
        const cx<T>* src = buf + f * GP + j;
#pragma unroll
        for (int t = 0; t < 16; ++t) v[s][t] = src[t * P::nb1];
      }
    }
    __syncthreads();
    pass1_store(v, buf);
    __syncthreads();
  }
  static __device__ __forceinline__ void pass2(cx<T>* buf, const cx<T>* twl) {
    constexpr int R = P::R2;
    cx<T> v[S2][R];
#pragma unroll
    for (int s = 0; s < S2; ++s) {
      const int u = (int)threadIdx.x + s * NT;
      if (u < FC * P::nb2) {
        const int f = u / P::nb2, j = u - f * P::nb2;
        const cx<T>* src = buf + f * GP + j + (j >> 4);
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
      const int u = (int)threadIdx.x + s * NT;
      if (u < FC * P::nb2) {
        const int f = u / P::nb2, j = u - f * P::nb2;
        cx<T>* d = buf + f * GP + (j >> 4) * (16 * R) + (j & 15);
#pragma unroll
        for (int t = 0; t < R; ++t) d[t * 16] = v[s][t];
      }
    }
    __syncthreads();
  }
  static __device__ __forceinline__ void pass3_regs(cx<T> (&v)[S3][P::R3], const cx<T>* buf, const cx<T>* twl) {
    constexpr int R = P::R3;
#pragma unroll
    for (int s = 0; s < S3; ++s) {
      const int u = (int)threadIdx.x + s * NT;
      if (u < FC * P::nb3) {
        const int f = u / P::nb3, j = u - f * P::nb3;
        const cx<T>* src = buf + f * GP + j;
#pragma unroll
        for (int t = 0; t < R; ++t) v[s][t] = src[t * P::nb3];
        const cx<T>* w = twl + P::tw3 + j;
#pragma unroll
        for (int t = 1; t < R; ++t) v[s][t] = cmul(v[s][t], w[(t - 1) * P::Ns3]);
        Dft<T, R>::run(v[s]);
      }
    }
  }

  template <int NL>
  static __device__ __forceinline__ int analysis(const FftArgsN<NL>& a, int l, int item, unsigned char* smem_raw) {
    cx<T>* buf = reinterpret_cast<cx<T>*>(smem_raw);
    cx<T>* twl = buf + FC * GP;
    const LevelDesc& L = a.lev[l];
    const int s0 = L.fft_item0, end = level_end(a, l), n = end - s0;
    const T* grid = static_cast<const T*>(a.src) + L.grid_off;
    T* ws = static_cast<T*>(a.dst) + L.ws_off;
    const T msc = (T)a.mscale;
    const int N = L.N, J = L.J, F = L.F, nfg = L.nfb;
    if (item >= end) return item;
    stage_twiddles(twl, static_cast<const cx<T>*>(L.tw));
    cx<T> v1[S1][16];
    auto load_rows = [&](int slot) __attribute__((always_inline)) {
      const int itm = xcd_map(slot - s0, n);
      const int jp = itm / nfg, fg = itm - jp * nfg;
      const bool eq = (J & 1) && (jp == (J >> 1));
      // uniform row bases plus a 32-bit lane offset (field and position)
      const char* gn = reinterpret_cast<const char*>(grid + ((long long)fg * FC * J + jp) * I);
      const char* gs = gn + (long long)(J - 1 - 2 * jp) * I * (int)sizeof(T);
#pragma unroll
      for (int s = 0; s < S1; ++s) {
        const int u = (int)threadIdx.x + s * NT;
        const int f = u / P::nb1, j = u - f * P::nb1;
        const unsigned lo = ((unsigned)f * (unsigned)(J * I) + (unsigned)j) * (unsigned)sizeof(T);
#pragma unroll
        for (int t = 0; t < 16; ++t) v1[s][t] = cx<T>{(T)0, (T)0};
        if (u < FC * P::nb1 && fg * FC + f < F) {
#pragma unroll
          for (int t = 0; t < 16; ++t)
            v1[s][t].x = *reinterpret_cast<const T*>(gn + t * P::nb1 * sizeof(T) + lo);
          if (!eq) {
#pragma unroll
            for (int t = 0; t < 16; ++t)
              v1[s][t].y = *reinterpret_cast<const T*>(gs + t * P::nb1 * sizeof(T) + lo);
          }
        }
      }
    };
    if constexpr (PF) load_rows(item);
    for (; item < end; item += gridDim.x) {
      const int itm = xcd_map(item - s0, n);
      const int jp = itm / nfg, fg = itm - jp * nfg;
      const bool eq = (J & 1) && (jp == (J >> 1));
      const T rscale = row_scale<T>(a, L, jp);
      const int next = item + (int)gridDim.x;
      if constexpr (!PF) load_rows(item);
      pass1_store(v1, buf);
      __syncthreads();
      if constexpr (PF)
        if (next < end) load_rows(next);
      pass2(buf, twl);
      {
        cx<T> v3[S3][P::R3];
        pass3_regs(v3, buf, twl);
        __syncthreads();
#pragma unroll
        for (int s = 0; s < S3; ++s) {
          const int u = (int)threadIdx.x + s * NT;
          if (u < FC * P::nb3) {
            const int f = u / P::nb3, j = u - f * P::nb3;
            cx<T>* d = buf + f * GP + j;
#pragma unroll
            for (int t = 0; t < P::R3; ++t) d[t * P::Ns3] = v3[s][t];
          }
        }
        __syncthreads();
      }
      T* wr = ws + (jp / SHT_K_PAD) * L.wjb + (long long)(jp % SHT_K_PAD) * 2 * L.Cp;
      const long long plane2 = L.wblk;
      const unsigned step = (unsigned)(plane2 * (long long)sizeof(T));
      const int units = (N + 1) * LV;
#pragma unroll 1
      for (int x = threadIdx.x; x < units; x += NT) {
        const int m = x / LV, f0 = (x - m * LV) * VW;
        const int fld = fg * FC + f0;
        if (fld >= F) continue;
        const T sc = m == 0 ? rscale : rscale * msc;
        typedef T TW __attribute__((ext_vector_type(2 * VW)));
        TW o, e;
#pragma unroll
        for (int q = 0; q < VW; ++q) {
          const cx<T>* z = buf + (f0 + q) * GP;
          const cx<T> Pm = z[m];
          cx<T> Q = z[m == 0 ? 0 : I - m];
          Q.y = -Q.y;  // conj Z^{I-m}
          const T h = (T)0.5;
          const cx<T> Xn = {h * (Pm.x + Q.x), h * (Pm.y + Q.y)};
          const cx<T> Xs = {h * (Pm.y - Q.y), -h * (Pm.x - Q.x)};
          cx<T> S = {sc * (Xn.x + Xs.x), sc * (Xn.y + Xs.y)};
          cx<T> A = {sc * (Xn.x - Xs.x), sc * (Xn.y - Xs.y)};
          if (m == 0) {
            S.y = (T)0;
            A.y = (T)0;
          }
          if (eq) A = cx<T>{(T)0, (T)0};
          e[2 * q] = S.x;
          e[2 * q + 1] = S.y;
          o[2 * q] = A.x;
          o[2 * q + 1] = A.y;
        }
        const int mw = __builtin_amdgcn_readfirstlane(m);
        char* wb = reinterpret_cast<char*>(wr + mw * plane2);
        const unsigned lo = (unsigned)(m - mw) * step + (unsigned)ws_col(L.wsh, 0, 2 * fld) * (unsigned)sizeof(T);
        *reinterpret_cast<TW*>(wb + lo) = e;
        *reinterpret_cast<TW*>(wb + lo + ((unsigned)sizeof(T) << L.wsh)) = o;
      }
      __syncthreads();
    }
    return item;
  }

  template <int NL>
  static __device__ __forceinline__ int synthesis(const FftArgsN<NL>& a, int l, int item, unsigned char* smem_raw) {
    typedef T TW __attribute__((ext_vector_type(2 * VW)));
    cx<T>* buf = reinterpret_cast<cx<T>*>(smem_raw);
    cx<T>* twl = buf + FC * GP;
    const LevelDesc& L = a.lev[l];
    const int s0 = L.fft_item0, end = level_end(a, l), n = end - s0;
    const T* ws = static_cast<const T*>(a.src) + L.ws_off;
    T* grid = static_cast<T*>(a.dst) + L.grid_off;
    const T msc = (T)a.mscale;
    const int N = L.N, J = L.J, F = L.F, nfg = L.nfb;
    const long long plane2 = L.wblk;
    const unsigned step = (unsigned)(plane2 * (long long)sizeof(T));
    TW pS[UM], pA[UM];
    auto load_ws = [&](int slot) __attribute__((always_inline)) {
      const int itm = xcd_map(slot - s0, n);
      const int jp = itm / nfg, fg = itm - jp * nfg;
      const int jb = jp / SHT_K_PAD;
      const T* w = ws + jb * L.wjb + (long long)(jp % SHT_K_PAD) * L.Cp + 2 * fg * FC;
      const long long odd = ws_odd(L.Jh, L.Cp, L.wblk, jb) * (long long)sizeof(T);
#pragma unroll
      for (int u = 0; u < UM; ++u) {
        const int x = (int)threadIdx.x + u * NT;
        const int m = x / LV, f0 = (x - m * LV) * VW;
        pS[u] = TW{};
        pA[u] = TW{};
        const int mw = __builtin_amdgcn_readfirstlane(m);
        const char* wb = reinterpret_cast<const char*>(w + mw * plane2);
        const unsigned lo = (unsigned)(m - mw) * step + (unsigned)(2 * f0 * sizeof(T));
        // rows below the first 128-latitude tile the Legendre synthesis
        // computes for this m (reduced transform) are zero
        if (m <= N && fg * FC + f0 < F && (!a.jstart || jp >= (a.jstart[L.m_base + m] & ~127))) {
          pS[u] = *reinterpret_cast<const TW*>(wb + lo);
          pA[u] = *reinterpret_cast<const TW*>(wb + odd + lo);
        }
      }
    };
    if (item >= end) return item;
    stage_twiddles(twl, static_cast<const cx<T>*>(L.tw));
    if constexpr (PF) load_ws(item);
    for (; item < end; item += gridDim.x) {
      const int itm = xcd_map(item - s0, n);
      const int jp = itm / nfg, fg = itm - jp * nfg;
      const bool eq = (J & 1) && (jp == (J >> 1));
      const T rscale = row_scale<T>(a, L, jp);
      const int next = item + (int)gridDim.x;
      if constexpr (!PF) load_ws(item);
#pragma unroll
      for (int f = 0; f < FC; ++f)  // the bins no unit fills: N < i < I - N
        for (int i = N + 1 + (int)threadIdx.x; i < I - N; i += NT) buf[f * GP + i] = cx<T>{(T)0, (T)0};
#pragma unroll
      for (int u = 0; u < UM; ++u) {
        const int x = (int)threadIdx.x + u * NT;
        const int m = x / LV, f0 = (x - m * LV) * VW;
        if (m <= N) {
          const T sc = m == 0 ? (T)1 : msc;
#pragma unroll
          for (int q = 0; q < VW; ++q) {
            const cx<T> S = {pS[u][2 * q], pS[u][2 * q + 1]}, A = {pA[u][2 * q], pA[u][2 * q + 1]};
            cx<T> Xn = {sc * (S.x + A.x), sc * (S.y + A.y)};
            cx<T> Xs = {sc * (S.x - A.x), sc * (S.y - A.y)};
            if (m == 0) {
              Xn.y = (T)0;
              Xs.y = (T)0;
            }
            // conj(Z), as in sht_fft.hip
            cx<T>* z = buf + (f0 + q) * GP;
            z[m] = cx<T>{Xn.x - Xs.y, -(Xn.y + Xs.x)};
            if (m > 0) z[I - m] = cx<T>{Xn.x + Xs.y, Xn.y - Xs.x};
          }
        }
      }
      __syncthreads();
      if constexpr (PF)
        if (next < end) load_ws(next);
      pass1_lds(buf);
      pass2(buf, twl);
      cx<T> v3[S3][P::R3];
      pass3_regs(v3, buf, twl);
      char* gn = reinterpret_cast<char*>(grid + ((long long)fg * FC * J + jp) * I);
      char* gs = gn + (long long)(J - 1 - 2 * jp) * I * (int)sizeof(T);
#pragma unroll
      for (int s = 0; s < S3; ++s) {
        const int u = (int)threadIdx.x + s * NT;
        const int f = u / P::nb3, j = u - f * P::nb3;
        const unsigned lo = ((unsigned)f * (unsigned)(J * I) + (unsigned)j) * (unsigned)sizeof(T);
        if (u < FC * P::nb3 && fg * FC + f < F) {
#pragma unroll
          for (int t = 0; t < P::R3; ++t)
            *reinterpret_cast<T*>(gn + t * P::Ns3 * sizeof(T) + lo) = rscale * v3[s][t].x;
          if (!eq) {
#pragma unroll
            for (int t = 0; t < P::R3; ++t)
              *reinterpret_cast<T*>(gs + t * P::Ns3 * sizeof(T) + lo) = -rscale * v3[s][t].y;
          }
        }
      }
      __syncthreads();
    }
    return item;
  }
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
// ahead.
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

}  // namespace sht

#endif  // SHT_GROUP_H_
