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

// NT: threads of an item
template <typename T, int NL>
static hipError_t any_shape(bool analysis, int NT, bool vec, const FftArgsN<NL>& a, size_t lds, int ncu,
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
  if constexpr (sizeof(T) == 4) {
    if (NT == 1024) return any_dir<T, 1024, true, 2>(analysis, a, lds, ncu, st);
  }
  if (a.lfc == 0) return NT == 256 ? go(N256{}, One{}) : go(N512{}, One{});
  return NT == 256 ? go(N256{}, VWT{}) : go(N512{}, VWT{});
}

template <typename T>
static hipError_t any_launch(bool analysis, const FftArgs& a0, int ncu, hipStream_t st) {
  constexpr int V = 16 / (int)sizeof(T);
  FftArgs a = a0;
  const AnyShape s = any_choice(sizeof(T), a.nlev, a.lev, ncu);
  const int fc = 1 << s.lfc;
  a.lfc = s.lfc;
  a.tw_lds = s.tw_lds;
  if (s.lds > kAnyMaxLds) return hipErrorInvalidValue;
  long long items = 0;
  for (int l = 0; l < a.nlev; ++l) {
    LevelDesc& L = a.lev[l];
    const int nv = s.vec ? any_nvec<V>(L.I) : L.I;
    L.ivm = nv > 1 ? 0xFFFFFFFFu / (unsigned)nv + 1u : 0u;
    L.nfb = (L.F + fc - 1) / fc;
    L.fft_item0 = (int)items;
    items += (long long)L.Jh * L.nfb;
  }
  if (items > 0x7fffffff) return hipErrorInvalidValue;
  a.nitems = (int)items;
  return a.nlev == 1 ? any_shape<T>(analysis, s.nt, s.vec, one_level(a), s.lds, ncu, st)
                     : any_shape<T>(analysis, s.nt, s.vec, a, s.lds, ncu, st);
}

int launch_zonal_any(bool dbl, bool analysis, const FftArgs& a, int ncu, void* stream) {
  hipStream_t st = static_cast<hipStream_t>(stream);
  return (int)(dbl ? any_launch<double>(analysis, a, ncu, st) : any_launch<float>(analysis, a, ncu, st));
}

}  // namespace sht
