// Device pieces shared by the zonal kernels: complex arithmetic, in-register
// DFTs of small lengths, and the mapping of workgroup slots to work items.
#ifndef SHT_DFT_H_
#define SHT_DFT_H_

#include <hip/hip_runtime.h>

#include <type_traits>
#include <utility>

#include "sht_internal.h"

namespace sht {

template <typename T>
struct cx {
  T x, y;
};

template <typename T>
__device__ __forceinline__ cx<T> cmul(cx<T> a, cx<T> b) {
  return {a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x};
}

template <typename T>
__device__ __forceinline__ cx<T> cadd(cx<T> a, cx<T> b) {
  return {a.x + b.x, a.y + b.y};
}

template <typename T>
__device__ __forceinline__ cx<T> csub(cx<T> a, cx<T> b) {
  return {a.x - b.x, a.y - b.y};
}

// multiply by -i
template <typename T>
__device__ __forceinline__ cx<T> mul_mi(cx<T> a) {
  return {a.y, -a.x};
}

// In-register DFT of length R with the forward sign exp(-2 pi i t k / R).
template <typename T, int R>
struct Dft;

template <typename T>
struct Dft<T, 2> {
  static __device__ __forceinline__ void run(cx<T>* v) {
    cx<T> a = v[0], b = v[1];
    v[0] = cadd(a, b);
    v[1] = csub(a, b);
  }
};

template <typename T>
struct Dft<T, 3> {
  static __device__ __forceinline__ void run(cx<T>* v) {
    const T h = (T)0.5;
    const T s = (T)0.86602540378443864676372317075293618;  // sin(2 pi / 3)
    cx<T> a = v[0], b = v[1], c = v[2];
    cx<T> sbc = cadd(b, c);
    cx<T> dbc = csub(b, c);
    cx<T> t1 = {a.x - h * sbc.x, a.y - h * sbc.y};
    // -i s (b - c)
    cx<T> t2 = {s * dbc.y, -s * dbc.x};
    v[0] = cadd(a, sbc);
    v[1] = cadd(t1, t2);
    v[2] = csub(t1, t2);
  }
};

template <typename T>
struct Dft<T, 4> {
  static __device__ __forceinline__ void run(cx<T>* v) {
    cx<T> a = v[0], b = v[1], c = v[2], d = v[3];
    cx<T> s0 = cadd(a, c), d0 = csub(a, c);
    cx<T> s1 = cadd(b, d), d1 = mul_mi(csub(b, d));
    v[0] = cadd(s0, s1);
    v[2] = csub(s0, s1);
    v[1] = cadd(d0, d1);
    v[3] = csub(d0, d1);
  }
};

template <typename T>
struct Dft<T, 8> {
  static __device__ __forceinline__ void run(cx<T>* v) {
    const T r = (T)0.70710678118654752440084436210484904;  // 1/sqrt(2)
    cx<T> e[4] = {v[0], v[2], v[4], v[6]};
    cx<T> o[4] = {v[1], v[3], v[5], v[7]};
    Dft<T, 4>::run(e);
    Dft<T, 4>::run(o);
    // o_k *= exp(-2 pi i k / 8)
    const cx<T> o1 = {r * (o[1].x + o[1].y), r * (o[1].y - o[1].x)};
    const cx<T> o2 = {o[2].y, -o[2].x};
    const cx<T> o3 = {r * (o[3].y - o[3].x), -r * (o[3].x + o[3].y)};
    v[0] = cadd(e[0], o[0]);
    v[4] = csub(e[0], o[0]);
    v[1] = cadd(e[1], o1);
    v[5] = csub(e[1], o1);
    v[2] = cadd(e[2], o2);
    v[6] = csub(e[2], o2);
    v[3] = cadd(e[3], o3);
    v[7] = csub(e[3], o3);
  }
};

template <typename T>
struct Dft<T, 5> {
  static __device__ __forceinline__ void run(cx<T>* v) {
    const T c1 = (T)0.30901699437494742410229341718281906;   // cos(2 pi/5)
    const T c2 = (T)-0.80901699437494742410229341718281906;  // cos(4 pi/5)
    const T s1 = (T)0.95105651629515357211643933337938214;   // sin(2 pi/5)
    const T s2 = (T)0.58778525229247312916870595463907277;   // sin(4 pi/5)
    cx<T> x0 = v[0];
    cx<T> p1 = cadd(v[1], v[4]), q1 = csub(v[1], v[4]);
    cx<T> p2 = cadd(v[2], v[3]), q2 = csub(v[2], v[3]);
    cx<T> r1 = {x0.x + c1 * p1.x + c2 * p2.x, x0.y + c1 * p1.y + c2 * p2.y};
    cx<T> r2 = {x0.x + c2 * p1.x + c1 * p2.x, x0.y + c2 * p1.y + c1 * p2.y};
    // i1 = s1 q1 + s2 q2, i2 = s2 q1 - s1 q2; y1 = r1 - i*i1, y4 = r1 + i*i1,
    // y2 = r2 - i*i2, y3 = r2 + i*i2
    cx<T> i1 = {s1 * q1.x + s2 * q2.x, s1 * q1.y + s2 * q2.y};
    cx<T> i2 = {s2 * q1.x - s1 * q2.x, s2 * q1.y - s1 * q2.y};
    v[0] = {x0.x + p1.x + p2.x, x0.y + p1.y + p2.y};
    v[1] = {r1.x + i1.y, r1.y - i1.x};
    v[4] = {r1.x - i1.y, r1.y + i1.x};
    v[2] = {r2.x + i2.y, r2.y - i2.x};
    v[3] = {r2.x - i2.y, r2.y + i2.x};
  }
};

// ---------------------------------------------------------------------------
// Composite in-register DFTs, R = R1 * R2 (Cooley-Tukey): R2 DFTs of length
// R1 over the inputs n = R2 n1 + n2, the internal twiddles
// exp(-2 pi i n2 k1 / R), then R1 DFTs of length R2; output index
// k = k1 + R1 k2.  The twiddles are compile-time constants.
// ---------------------------------------------------------------------------
constexpr double kTwoPi = 6.283185307179586476925286766559005768;

// sin(x) for |x| <= pi/2 by its Taylor series (accurate to double rounding)
constexpr double csin_small(double x) {
  double x2 = x * x, term = x, sum = x;
  for (int k = 1; k < 14; ++k) {
    term *= -x2 / ((2.0 * k) * (2.0 * k + 1.0));
    sum += term;
  }
  return sum;
}

// sin(2 pi e / R) and cos(2 pi e / R) with exact integer range reduction
constexpr double csin2pi(int e, int R) {
  e %= R;
  if (e < 0) e += R;
  // reduce to the first half turn by symmetry: sin(2 pi - x) = -sin(x)
  if (2 * e > R) return -csin2pi(R - e, R);
  // x = 2 pi e / R in [0, pi]; sin(x) = sin(pi - x)
  if (4 * e > R) return csin_small(kTwoPi * (double)(R - 2 * e) / (2.0 * R));
  return csin_small(kTwoPi * (double)e / (double)R);
}

constexpr double ccos2pi(int e, int R) { return csin2pi(4 * e + R, 4 * R); }

// Calls f(integral_constant<int, i>) for i = 0..N-1, so that f can form
// constant expressions from i.
template <class F, int... Is>
__device__ __forceinline__ void static_for_impl(F& f, std::integer_sequence<int, Is...>) {
  (f(std::integral_constant<int, Is>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for(F f) {
  static_for_impl(f, std::make_integer_sequence<int, N>{});
}

template <typename T, int R1, int R2>
struct DftCT {
  static constexpr int R = R1 * R2;
  static __device__ __forceinline__ void run(cx<T>* v) {
    cx<T> y[R2][R1];
    static_for<R2>([&](auto n2c) {
      constexpr int n2 = decltype(n2c)::value;
      cx<T> t[R1];
#pragma unroll
      for (int n1 = 0; n1 < R1; ++n1) t[n1] = v[R2 * n1 + n2];
      Dft<T, R1>::run(t);
      static_for<R1>([&](auto k1c) {
        constexpr int k1 = decltype(k1c)::value;
        if constexpr (n2 == 0 || k1 == 0) {
          y[n2][k1] = t[k1];
        } else {
          constexpr T c = (T)ccos2pi(n2 * k1, R), sn = (T)-csin2pi(n2 * k1, R);
          y[n2][k1] = cx<T>{t[k1].x * c - t[k1].y * sn, t[k1].x * sn + t[k1].y * c};
        }
      });
    });
#pragma unroll
    for (int k1 = 0; k1 < R1; ++k1) {
      cx<T> t[R2];
#pragma unroll
      for (int n2 = 0; n2 < R2; ++n2) t[n2] = y[n2][k1];
      Dft<T, R2>::run(t);
#pragma unroll
      for (int k2 = 0; k2 < R2; ++k2) v[k1 + R1 * k2] = t[k2];
    }
  }
};

template <typename T>
struct Dft<T, 6> : DftCT<T, 3, 2> {};
template <typename T>
struct Dft<T, 9> : DftCT<T, 3, 3> {};
template <typename T>
struct Dft<T, 10> : DftCT<T, 5, 2> {};
template <typename T>
struct Dft<T, 12> : DftCT<T, 4, 3> {};
template <typename T>
struct Dft<T, 15> : DftCT<T, 5, 3> {};
template <typename T>
struct Dft<T, 16> : DftCT<T, 4, 4> {};

// q = floor(j / d) for 0 <= j < 2^16 and 2 <= d <= 4096, with
// magic = floor((2^32 - 1) / d) + 1 = ceil(2^32 / d): the excess
// j (magic d - 2^32) < 2^16 d stays below 2^32.
__device__ __forceinline__ int fastdiv(int j, unsigned magic) {
  return (int)__umulhi((unsigned)j, magic);
}

template <typename T>
struct Vec16;
template <>
struct Vec16<float> {
  typedef float type __attribute__((ext_vector_type(4)));
};
template <>
struct Vec16<double> {
  typedef double type __attribute__((ext_vector_type(2)));
};

template <int NL>
__device__ __forceinline__ int level_of(const FftArgsN<NL>& a, int item) {
  if (NL == 1) return 0;
  int l = 0;
  while (l + 1 < a.nlev && item >= a.lev[l + 1].fft_item0) ++l;
  return l;
}

// One past the last work item (slot) of level l.
template <int NL>
__device__ __forceinline__ int level_end(const FftArgsN<NL>& a, int l) {
  if (NL == 1) return a.nitems;
  return l + 1 < a.nlev ? a.lev[l + 1].fft_item0 : a.nitems;
}

// Workgroup b runs on XCD b mod 8 and walks the slots b, b + G, ...
// (G = gridDim.x, a multiple of 8 on a full device).  The slots of a level
// are a contiguous range; within it, local slot i is mapped to the level's
// list position x R' + k (x = i mod 8, k = i / 8, R' the length of the
// x-th eighth of the level's list): the workgroups of one XCD work through
// one contiguous eighth of every level, so the field blocks of one latitude
// pair run on one XCD at about the same time and fill whole workspace lines
// in its L2, and every XCD gets the same share of each level.  The map is a
// permutation of [0, n).
__device__ __forceinline__ int xcd_map(int i, int n) {
  const int x = i & 7, k = i >> 3;
  const int R = n >> 3, rem = n & 7;
  return x * R + (x < rem ? x : rem) + k;
}

template <typename T, int NL>
__device__ __forceinline__ T row_scale(const FftArgsN<NL>& a, const LevelDesc& L, int jp) {
  T r = (T)1;
  if (a.use_w) r = (T)L.wrow[jp];
  if (a.use_inv_I) r = (T)((double)r / (double)L.I);
  return r;
}

}  // namespace sht

#endif  // SHT_DFT_H_
