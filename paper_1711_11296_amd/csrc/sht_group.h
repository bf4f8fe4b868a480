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
// compute phases.  GroupShape (sht_zonal_rule.h) has the shapes and what they measured.
#ifndef SHT_GROUP_H_
#define SHT_GROUP_H_

#include <hip/hip_runtime.h>

#include "sht_any.h"
#include "sht_dft.h"
#include "sht_internal.h"
#include "sht_zonal_rule.h"

namespace sht {

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
    // rows below the first 128-latitude tile the Legendre synthesis computes
    // for a wavenumber (reduced transform) are zero; a thread's wavenumbers are
    // the same in every item, and read per item the limits precede the runs in
    // a chain of two loads (T959 FP32 reduced 690 -> 635 us).  The kernels whose
    // registers are full without them read them per item all the same (I = 1600
    // FP32, 641 rows, 64 fields, full transform: held 148 us, per item 124; the
    // one launch over several levels 4-12 % longer)
    constexpr bool LIM = NL == 1 && !(sizeof(T) == 4 && (I == 1600 || I == 3600));
    int lim[UM];
    if constexpr (LIM)
#pragma unroll
      for (int u = 0; u < UM; ++u) {
        const int m = ((int)threadIdx.x + u * NT) / LV;
        lim[u] = m > N ? 0x7fffffff : a.jstart ? a.jstart[L.m_base + m] & ~127 : 0;
      }
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
        if (LIM ? jp >= lim[u] && fg * FC + f0 < F
                : m <= N && fg * FC + f0 < F && (!a.jstart || jp >= (a.jstart[L.m_base + m] & ~127))) {
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

}  // namespace sht

#endif  // SHT_GROUP_H_
