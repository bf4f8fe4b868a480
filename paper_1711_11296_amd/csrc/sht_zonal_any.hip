// Launches of the any-length zonal kernels (sht_any.h).

#include <hip/hip_runtime.h>

#include <type_traits>

#include "sht_any.h"
#include "sht_internal.h"

namespace sht {

// waves per SIMD the kernels are compiled for
template <typename T>
constexpr int any_wpe() {
  return sizeof(T) == 4 ? 4 : 2;
}

template <typename T, int NT, bool VEC, int VW, int NL>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(any_wpe<T>()))) void k_zonal_any_analysis(const FftArgsN<NL> a) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  any_analysis_run<T, NT, VEC, VW>(a, blockIdx.x, a.nitems, smem_raw);
}

template <typename T, int NT, bool VEC, int VW, int NL>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(any_wpe<T>()))) void k_zonal_any_synthesis(const FftArgsN<NL> a) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  any_synthesis_run<T, NT, VEC, VW>(a, blockIdx.x, a.nitems, smem_raw);
}

// ---------------------------------------------------------------------------
// launcher
// ---------------------------------------------------------------------------
constexpr size_t kAnyMaxLds = 160 * 1024;

template <auto Kernel, class A>
static hipError_t any_go(const A& a, int NT, int wpe, size_t lds, int ncu, hipStream_t st) {
  static size_t done = 0;
  if (lds > 65536 && lds > done) {
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(Kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                              (int)kAnyMaxLds);
    done = kAnyMaxLds;
  }
  // persistent workgroups, as many as fit at the kernels' waves per SIMD
  int per_cu = (int)(kAnyMaxLds / lds);
  per_cu = per_cu < wpe * 256 / NT ? per_cu : wpe * 256 / NT;
  per_cu = per_cu < 1 ? 1 : per_cu;
  const int nwg = ncu * per_cu < a.nitems ? ncu * per_cu : a.nitems;
  hipLaunchKernelGGL(Kernel, dim3(nwg), dim3(NT), lds, st, a);
  return hipGetLastError();
}

template <typename T, int NT, bool VEC, int VW, int NL>
static hipError_t any_dir(bool analysis, const FftArgsN<NL>& a, size_t lds, int ncu, hipStream_t st) {
  return analysis ? any_go<k_zonal_any_analysis<T, NT, VEC, VW, NL>>(a, NT, any_wpe<T>(), lds, ncu, st)
                  : any_go<k_zonal_any_synthesis<T, NT, VEC, VW, NL>>(a, NT, any_wpe<T>(), lds, ncu, st);
}

template <typename T, int NL>
static hipError_t any_shape(bool analysis, bool small, bool vec, const FftArgsN<NL>& a, size_t lds, int ncu,
                            hipStream_t st) {
  auto go = [&](auto nt, auto vw) {
    constexpr int NT = decltype(nt)::value, VW = decltype(vw)::value;
    return vec ? any_dir<T, NT, true, VW>(analysis, a, lds, ncu, st)
               : any_dir<T, NT, false, VW>(analysis, a, lds, ncu, st);
  };
  using N256 = std::integral_constant<int, 256>;
  using N512 = std::integral_constant<int, 512>;
  using One = std::integral_constant<int, 1>;
  using VWT = std::integral_constant<int, sizeof(T) == 4 ? 2 : 1>;
  if (a.lfc == 0) return small ? go(N256{}, One{}) : go(N512{}, One{});
  return small ? go(N256{}, VWT{}) : go(N512{}, VWT{});
}

template <typename T>
static hipError_t any_launch(bool analysis, const FftArgs& a0, int ncu, hipStream_t st) {
  constexpr int E = AnyCap<T>::E, V = 16 / (int)sizeof(T);
  FftArgs a = a0;
  int maxI = 0, maxR = 0, maxN = 0, maxIP = 0, maxF = 0;  // maxR: whole vectors
  bool vec = true;
  for (int l = 0; l < a.nlev; ++l) {
    const LevelDesc& L = a.lev[l];
    maxI = L.I > maxI ? L.I : maxI;
    maxN = L.N > maxN ? L.N : maxN;
    maxF = L.F > maxF ? L.F : maxF;
    const int ip = any_stride(L);
    maxIP = ip > maxIP ? ip : maxIP;
    const int r = any_nvec<V>(L.I) * V;
    maxR = r > maxR ? r : maxR;
    vec = vec && L.I >= V;
  }
  // fields per item: as many as a workspace run holds, as long as two
  // workgroups share a compute unit's LDS, no group is mostly empty and the
  // device has an item per compute unit (T85 with 7 fields: 28 us a pair with
  // two per unit, one field each, 24 with one)
  auto lds_of = [&](int fc) { return (size_t)((size_t)fc * maxIP + maxI) * sizeof(cx<T>); };
  auto items_of = [&](int fc) {
    long long n = 0;
    for (int l = 0; l < a.nlev; ++l) n += (long long)a.lev[l].Jh * ((a.lev[l].F + fc - 1) / fc);
    return n;
  };
  int lfc = sizeof(T) == 4 ? 3 : 2;
  while (lfc > 0 && ((1 << lfc) * (long long)maxR > 512LL * E || (1 << lfc) * (maxN + 1LL) > 256LL * E ||
                     lds_of(1 << lfc) > kAnyMaxLds / 2 || (1 << (lfc - 1)) >= maxF || items_of(1 << lfc) < ncu))
    --lfc;
  const int fc = 1 << lfc;
  const bool small = fc * (long long)maxR <= 256LL * E && fc * (maxN + 1LL) <= 128LL * E;
  a.lfc = lfc;
  a.tw_lds = (fc * maxIP + 1) & ~1;
  const size_t lds = ((size_t)a.tw_lds + maxI) * sizeof(cx<T>);
  if (lds > kAnyMaxLds) return hipErrorInvalidValue;
  long long items = 0;
  for (int l = 0; l < a.nlev; ++l) {
    LevelDesc& L = a.lev[l];
    const int nv = vec ? any_nvec<V>(L.I) : L.I;
    L.ivm = nv > 1 ? 0xFFFFFFFFu / (unsigned)nv + 1u : 0u;
    L.nfb = (L.F + fc - 1) / fc;
    L.fft_item0 = (int)items;
    items += (long long)L.Jh * L.nfb;
  }
  if (items > 0x7fffffff) return hipErrorInvalidValue;
  a.nitems = (int)items;
  return a.nlev == 1 ? any_shape<T>(analysis, small, vec, one_level(a), lds, ncu, st)
                     : any_shape<T>(analysis, small, vec, a, lds, ncu, st);
}

int launch_zonal_any(bool dbl, bool analysis, const FftArgs& a, int ncu, void* stream) {
  hipStream_t st = static_cast<hipStream_t>(stream);
  return (int)(dbl ? any_launch<double>(analysis, a, ncu, st) : any_launch<float>(analysis, a, ncu, st));
}

}  // namespace sht
