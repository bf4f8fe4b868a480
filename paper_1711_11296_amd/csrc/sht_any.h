// Zonal stage for lengths without a compile-time plan: the transform, fold
// and workspace layouts are those of sht_fft.hip; the radices, strides and
// the number of fields per work item are values of the launch.
//
// Work item = (mirror row pair, group of FC fields), FC a power of two.  The
// FC complex sequences z = x_north + i x_south lie side by side in LDS; each
// Stockham pass deals the butterflies of all FC sequences to the threads, so
// that short rows fill a workgroup too, and between the passes nothing is
// held in registers: the fold (or its inverse) reads (writes) the sequences
// in LDS and stores (loads) 16-byte pieces of the workspace runs directly.
// Rows move as 16-byte vectors of any length: the last vector of a row starts
// early enough to end with it (its first values are its neighbour's too), and
// rows need only be aligned to their elements.  The next
// item's rows (runs) are fetched into registers while the current item is
// transformed.
//
// Passes: the radices 2..16 of factor_radices, at most three for nearly
// every length.  The first pass stores its radix-R blocks with a pitch of
// R + 1 where R is even, so that the lanes' stores fall on distinct banks;
// the second pass reads that layout; later ones the natural order.
// Twiddles of pass p are staged in LDS as [t - 1][k].
//
// Bound: HBM for long batches, the chain of barriers for small ones.  The
// kernels these replaced ran the radices 8/4/2/3/5 (four or five passes),
// gave the threads of a workgroup the butterflies of one field (64 of 256
// threads busy at I = 512 in FP64) and walked all 8 (4) fields of a block
// whether they existed or not.  Measured on one box, analysis / synthesis,
// before and after: I = 1280, 640 rows, 40 fields FP32 155 / 151 -> 76 / 88
// us; I = 720, 479 rows, 100 fields 106 / 102 -> 75 / 72 us; I = 256, 171
// rows, 7 fields 17.0 / 15.3 -> 9.6 / 9.6 us; FP64 I = 1024, 959 rows, 32
// fields 205 / 191 -> 146 / 182 us.

#ifndef SHT_ANY_H_
#define SHT_ANY_H_

#include <hip/hip_runtime.h>

#include "sht_dft.h"
#include "sht_internal.h"
#include "sht_zonal_rule.h"

namespace sht {

// Complex values per thread.  (FP32: a pass then holds at most 20 complex
// values and the prefetch 24 floats, compiled for 4 waves per SIMD; FP64 takes
// the registers of 2.  With
// rows in vectors the single-level FP32 synthesis spills 8 registers with
// groups of 2 fields or more and 37 with single fields, the analysis none;
// with scalar rows, which only lengths below a vector take, 30 to 97.  The
// several-level and the FP64 kernels spill none.)
template <typename T>
struct AnyCap {
  static constexpr int E = any_values(sizeof(T));
};

template <typename T, int NT, int R>
__device__ __forceinline__ void any_pass(cx<T>* buf, const cx<T>* tw, int IP, int nfc, int p, int nb, int Ns,
                                         unsigned mnb, unsigned mns, bool padded) {
  constexpr int S = (AnyCap<T>::E + R - 1) / R;
  const int total = nfc * nb;
  const bool inpad = p == 1 && padded;
  const int istr = inpad ? nb + nb / Ns : nb;
  cx<T> v[S][R];
  int dst[S];
#pragma unroll
  for (int s = 0; s < S; ++s) {
    const int u = (int)threadIdx.x + s * NT;
    dst[s] = -1;
    if (u < total) {
      const int f = nb > 1 ? fastdiv(u, mnb) : u;
      const int j = u - f * nb;
      int q = j, k = 0;
      if (p > 0) {
        q = fastdiv(j, mns);
        k = j - q * Ns;
      }
      const cx<T>* src = buf + f * IP + j + (inpad ? q : 0);
#pragma unroll
      for (int t = 0; t < R; ++t) v[s][t] = src[t * istr];
      if (p > 0) {
        const cx<T>* w = tw + k;
#pragma unroll
        for (int t = 1; t < R; ++t) v[s][t] = cmul(v[s][t], w[(t - 1) * Ns]);
      }
      Dft<T, R>::run(v[s]);
      dst[s] = f * IP + (p == 0 ? (padded ? R + 1 : R) * j : q * (Ns * R) + k);
    }
  }
  __syncthreads();
#pragma unroll
  for (int s = 0; s < S; ++s)
    if (dst[s] >= 0) {
      cx<T>* d = buf + dst[s];
#pragma unroll
      for (int t = 0; t < R; ++t) d[t * Ns] = v[s][t];
    }
  __syncthreads();
}

// The level's FFTs of the FC sequences in buf, natural order in and out.
template <typename T, int NT>
__device__ __forceinline__ void any_fft(cx<T>* buf, const cx<T>* tw, const LevelDesc& L, int IP, int nfc) {
  const bool padded = L.nrad > 1 && L.rad[0] % 2 == 0;
  for (int p = 0; p < L.nrad; ++p) {
    const int R = L.rad[p], Ns = L.pns[p], nb = L.pnb[p];
    const unsigned mnb = L.pbm[p], mns = L.pmag[p];
#define SHT_ANY_PASS(r) \
  case r: any_pass<T, NT, r>(buf, tw, IP, nfc, p, nb, Ns, mnb, mns, padded); break;
    switch (R) {
      SHT_ANY_PASS(2)
      SHT_ANY_PASS(3)
      SHT_ANY_PASS(4)
      SHT_ANY_PASS(5)
      SHT_ANY_PASS(6)
      SHT_ANY_PASS(8)
      SHT_ANY_PASS(9)
      SHT_ANY_PASS(10)
      SHT_ANY_PASS(12)
      SHT_ANY_PASS(15)
      default: any_pass<T, NT, 16>(buf, tw, IP, nfc, p, nb, Ns, mnb, mns, padded); break;
    }
#undef SHT_ANY_PASS
    if (p > 0) tw += (R - 1) * Ns;
  }
}

template <typename T, int NT>
__device__ __forceinline__ void any_twiddles(cx<T>* tw, const LevelDesc& L) {
  const cx<T>* g = static_cast<const cx<T>*>(L.tw);
  int o = 0;
  for (int p = 1; p < L.nrad; ++p) {
    const int Ns = L.pns[p], n = (L.rad[p] - 1) * Ns, step = L.ptw[p];
    const unsigned mns = L.pmag[p];
    for (int x = threadIdx.x; x < n; x += NT) {
      const int t = fastdiv(x, mns), k = x - t * Ns;
      tw[o + x] = g[(t + 1) * k * step];
    }
    o += n;
  }
}

struct AnyItem {
  int l, jp, fg, js;
  bool eq;
};

template <int NL>
__device__ __forceinline__ AnyItem any_item(const FftArgsN<NL>& a, int slot) {
  AnyItem it;
  it.l = level_of(a, slot);
  const LevelDesc& L = a.lev[NL == 1 ? 0 : it.l];
  const int local = xcd_map(slot - L.fft_item0, level_end(a, it.l) - L.fft_item0);
  it.jp = local / L.nfb;
  it.fg = local - it.jp * L.nfb;
  it.eq = (L.J & 1) && it.jp == (L.J >> 1);
  it.js = L.J - 1 - it.jp;
  return it;
}

// The rows of FC fields as vectors of V values, aligned like T (the hardware
// takes such vector accesses): unit x = (field, vector).
template <typename T, int V>
struct AnyVec {
  typedef T vec __attribute__((ext_vector_type(V)));
  typedef vec type __attribute__((aligned(sizeof(T))));
};
template <typename T>
struct AnyVec<T, 1> {
  typedef T type;
};

template <typename T, int V>
__device__ __forceinline__ T any_get(const typename AnyVec<T, V>::type& v, int e) {
  if constexpr (V == 1)
    return v;
  else
    return v[e];
}

// analysis: grid [F][J][I] -> workspace S/A.  VEC: rows as 16-byte vectors
// (I at least one vector);
// VW: fields per workspace piece (2 in FP32 with FC >= 2: 16 bytes).
// The slots item, item + G, ... below `end` (any levels); returns the first
// slot past them.  Every thread of the workgroup calls it alike.
template <typename T, int NT, bool VEC, int VW, int NL>
__device__ __forceinline__ int any_analysis_run(const FftArgsN<NL>& a, int item, int end, unsigned char* smem_raw) {
  constexpr int E = AnyCap<T>::E, V = VEC ? 16 / (int)sizeof(T) : 1, LU = E / V;
  typedef typename AnyVec<T, V>::type TV;
  cx<T>* buf = reinterpret_cast<cx<T>*>(smem_raw);
  cx<T>* twl = buf + a.tw_lds;
  const T* grid0 = static_cast<const T*>(a.src);
  T* ws0 = static_cast<T*>(a.dst);
  const T msc = (T)a.mscale;
  const int lfc = a.lfc, FC = 1 << lfc;

  TV pn[LU], ps[LU];
  auto load_rows = [&](int slot) __attribute__((always_inline)) {
    const AnyItem it = any_item(a, slot);
    const LevelDesc& L = a.lev[NL == 1 ? 0 : it.l];
    const int nv = any_nvec<V>(L.I), F = L.F - it.fg * FC;  // fields of this group that exist
    const unsigned mv = L.ivm;
    const T* rn = grid0 + L.grid_off + ((long long)it.fg * FC * L.J + it.jp) * L.I;
    const T* rs = grid0 + L.grid_off + ((long long)it.fg * FC * L.J + it.js) * L.I;
    const long long fs = (long long)L.J * L.I;
#pragma unroll
    for (int u = 0; u < LU; ++u) {
      const int x = (int)threadIdx.x + u * NT;
      const int f = nv > 1 ? fastdiv(x, mv) : x, i = any_first<V>(x - f * nv, L.I);
      pn[u] = TV{};
      ps[u] = TV{};
      if (f < FC && f < F) {
        pn[u] = *reinterpret_cast<const TV*>(rn + f * fs + i);
        if (!it.eq) ps[u] = *reinterpret_cast<const TV*>(rs + f * fs + i);
      }
    }
  };

  if (item >= end) return item;
  load_rows(item);
  int lcur = -1;
  for (; item < end; item += gridDim.x) {
    const AnyItem it = any_item(a, item);
    const LevelDesc& L = a.lev[NL == 1 ? 0 : it.l];
    const int I = L.I, N = L.N, IP = any_stride(L);
    if (it.l != lcur) {
      any_twiddles<T, NT>(twl, L);  // (the barrier at the end of an item precedes it)
      lcur = it.l;
    }
    {
      const int nv = any_nvec<V>(I);
      const unsigned mv = L.ivm;
#pragma unroll
      for (int u = 0; u < LU; ++u) {
        const int x = (int)threadIdx.x + u * NT;
        const int f = nv > 1 ? fastdiv(x, mv) : x, i = any_first<V>(x - f * nv, I);
        if (f < FC) {
          cx<T>* d = buf + f * IP + i;
#pragma unroll
          for (int e = 0; e < V; ++e) d[e] = cx<T>{any_get<T, V>(pn[u], e), any_get<T, V>(ps[u], e)};
        }
      }
    }
    __syncthreads();
    if (item + (int)gridDim.x < end) load_rows(item + (int)gridDim.x);
    any_fft<T, NT>(buf, twl, L, IP, FC);

    // fold: unit = (wavenumber, VW fields)
    const T rscale = row_scale<T>(a, L, it.jp);
    T* ws = ws0 + L.ws_off + (it.jp / SHT_K_PAD) * L.wjb + (long long)(it.jp % SHT_K_PAD) * 2 * L.Cp;
    const long long region = L.wblk;
    constexpr int LVW = VW == 2 ? 1 : 0;
    const int units = (N + 1) << (lfc - LVW);
    for (int x = threadIdx.x; x < units; x += NT) {
      const int m = x >> (lfc - LVW), f0 = (x - (m << (lfc - LVW))) * VW;
      const int fld = it.fg * FC + f0;
      if (fld >= L.F) continue;
      const T sc = m == 0 ? rscale : rscale * msc;
      T oS[2 * VW], oA[2 * VW];
#pragma unroll
      for (int q = 0; q < VW; ++q) {
        const cx<T>* z = buf + (f0 + q) * IP;
        const cx<T> P = z[m];
        cx<T> Q = z[m == 0 ? 0 : I - m];
        Q.y = -Q.y;  // conj Z^{I-m}
        const T h = (T)0.5;
        const cx<T> Xn = {h * (P.x + Q.x), h * (P.y + Q.y)};
        const cx<T> Xs = {h * (P.y - Q.y), -h * (P.x - Q.x)};
        cx<T> S = {sc * (Xn.x + Xs.x), sc * (Xn.y + Xs.y)};
        cx<T> A = {sc * (Xn.x - Xs.x), sc * (Xn.y - Xs.y)};
        if (m == 0) {
          S.y = (T)0;
          A.y = (T)0;
        }
        if (it.eq) A = cx<T>{(T)0, (T)0};
        oS[2 * q] = S.x;
        oS[2 * q + 1] = S.y;
        oA[2 * q] = A.x;
        oA[2 * q + 1] = A.y;
      }
      T* d = ws + m * region + ws_col(L.wsh, 0, 2 * fld);
      typedef T TW __attribute__((ext_vector_type(2 * VW)));
      TW s, o;
#pragma unroll
      for (int e = 0; e < 2 * VW; ++e) {
        s[e] = oS[e];
        o[e] = oA[e];
      }
      *reinterpret_cast<TW*>(d) = s;
      *reinterpret_cast<TW*>(d + (1 << L.wsh)) = o;
    }
    __syncthreads();
  }
  return item;
}

// synthesis: workspace S/A -> grid [F][J][I]
template <typename T, int NT, bool VEC, int VW, int NL>
__device__ __forceinline__ int any_synthesis_run(const FftArgsN<NL>& a, int item, int end, unsigned char* smem_raw) {
  constexpr int E = AnyCap<T>::E, V = VEC ? 16 / (int)sizeof(T) : 1, LU = E / V, UM = E / (2 * VW);
  typedef typename AnyVec<T, V>::type TV;
  typedef T TW __attribute__((ext_vector_type(2 * VW)));
  cx<T>* buf = reinterpret_cast<cx<T>*>(smem_raw);
  cx<T>* twl = buf + a.tw_lds;
  const T* ws0 = static_cast<const T*>(a.src);
  T* grid0 = static_cast<T*>(a.dst);
  const T msc = (T)a.mscale;
  constexpr int LVW = VW == 2 ? 1 : 0;
  const int lfc = a.lfc, FC = 1 << lfc;

  TW pS[UM], pA[UM];
  // rows below the first 128-latitude tile the Legendre synthesis computes for
  // a wavenumber (reduced transform) are zero; with one level a thread's
  // wavenumbers are the same in every item
  int lim[UM];
  if constexpr (NL == 1)
#pragma unroll
    for (int u = 0; u < UM; ++u) {
      const int m = ((int)threadIdx.x + u * NT) >> (lfc - LVW);
      lim[u] = m > a.lev[0].N ? 0x7fffffff : a.jstart ? a.jstart[a.lev[0].m_base + m] & ~127 : 0;
    }
  auto load_ws = [&](int slot) __attribute__((always_inline)) {
    const AnyItem it = any_item(a, slot);
    const LevelDesc& L = a.lev[NL == 1 ? 0 : it.l];
    const int jb = it.jp / SHT_K_PAD;
    const T* ws = ws0 + L.ws_off + jb * L.wjb + (long long)(it.jp % SHT_K_PAD) * L.Cp + 2 * it.fg * FC;
    const long long region = L.wblk, odd = ws_odd(L.Jh, L.Cp, L.wblk, jb);
#pragma unroll
    for (int u = 0; u < UM; ++u) {
      const int x = (int)threadIdx.x + u * NT;
      const int m = x >> (lfc - LVW), f0 = (x - (m << (lfc - LVW))) * VW;
      pS[u] = TW{};
      pA[u] = TW{};
      if (NL == 1 ? it.jp >= lim[u] && it.fg * FC + f0 < L.F
                  : m <= L.N && it.fg * FC + f0 < L.F && (!a.jstart || it.jp >= (a.jstart[L.m_base + m] & ~127))) {
        const T* s = ws + m * region + 2 * f0;
        pS[u] = *reinterpret_cast<const TW*>(s);
        pA[u] = *reinterpret_cast<const TW*>(s + odd);
      }
    }
  };

  if (item >= end) return item;
  load_ws(item);
  int lcur = -1;
  for (; item < end; item += gridDim.x) {
    const AnyItem it = any_item(a, item);
    const LevelDesc& L = a.lev[NL == 1 ? 0 : it.l];
    const int I = L.I, N = L.N, IP = any_stride(L);
    if (it.l != lcur) {
      any_twiddles<T, NT>(twl, L);
      lcur = it.l;
    }
    // zero the bins no unit fills: N < i < I - N
    for (int f = 0; f < FC; ++f)
      for (int i = N + 1 + (int)threadIdx.x; i < I - N; i += NT) buf[f * IP + i] = cx<T>{(T)0, (T)0};
#pragma unroll
    for (int u = 0; u < UM; ++u) {
      const int x = (int)threadIdx.x + u * NT;
      const int m = x >> (lfc - LVW), f0 = (x - (m << (lfc - LVW))) * VW;
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
          cx<T>* z = buf + (f0 + q) * IP;
          z[m] = cx<T>{Xn.x - Xs.y, -(Xn.y + Xs.x)};
          if (m > 0) z[I - m] = cx<T>{Xn.x + Xs.y, Xn.y - Xs.x};
        }
      }
    }
    __syncthreads();
    if (item + (int)gridDim.x < end) load_ws(item + (int)gridDim.x);
    any_fft<T, NT>(buf, twl, L, IP, FC);

    const T rscale = row_scale<T>(a, L, it.jp);
    const int nv = any_nvec<V>(I), F = L.F - it.fg * FC;
    const unsigned mv = L.ivm;
    T* rn = grid0 + L.grid_off + ((long long)it.fg * FC * L.J + it.jp) * I;
    T* rs = grid0 + L.grid_off + ((long long)it.fg * FC * L.J + it.js) * I;
    const long long fs = (long long)L.J * I;
#pragma unroll
    for (int u = 0; u < LU; ++u) {
      const int x = (int)threadIdx.x + u * NT;
      const int f = nv > 1 ? fastdiv(x, mv) : x, i = any_first<V>(x - f * nv, I);
      if (f < FC && f < F) {
        const cx<T>* z = buf + f * IP + i;
        TV n, s;
        if constexpr (V == 1) {
          n = rscale * z[0].x;
          s = -rscale * z[0].y;
        } else {
#pragma unroll
          for (int e = 0; e < V; ++e) {
            n[e] = rscale * z[e].x;
            s[e] = -rscale * z[e].y;
          }
        }
        *reinterpret_cast<TV*>(rn + f * fs + i) = n;
        if (!it.eq) *reinterpret_cast<TV*>(rs + f * fs + i) = s;
      }
    }
    __syncthreads();
  }
  return item;
}


}  // namespace sht

#endif  // SHT_ANY_H_
