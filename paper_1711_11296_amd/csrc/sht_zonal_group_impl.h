// Launches of the group kernels (sht_group.h) of one element type and
// direction: SHT_GROUP_T, SHT_GROUP_ANA and SHT_GROUP_LAUNCH are set by the
// including file.

#include <hip/hip_runtime.h>

#include "sht_group.h"
#include "sht_internal.h"

namespace sht {

namespace {

template <typename T, int I, bool ANA>
__global__ __launch_bounds__((GroupShape<T, I, ANA>::NT))
    __attribute__((amdgpu_waves_per_eu(GroupShape<T, I, ANA>::WPE))) void k_zonal_group(const FftArgs1 a) {
  using S = GroupShape<T, I, ANA>;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  if constexpr (ANA)
    Grp<T, typename S::P, S::NT, S::FC, S::PF>::analysis(a, 0, blockIdx.x, smem_raw);
  else
    Grp<T, typename S::P, S::NT, S::FC, S::PF>::synthesis(a, 0, blockIdx.x, smem_raw);
}

template <typename T, int I, bool ANA>
int go(const FftArgs1& a0, int ncu, hipStream_t st) {
  using S = GroupShape<T, I, ANA>;
  using G = Grp<T, typename S::P, S::NT, S::FC, S::PF>;
  constexpr size_t lds = G::lds(), most = 160 * 1024;
  static_assert(lds <= most, "one workgroup's LDS");
  FftArgs1 a = a0;
  LevelDesc& L = a.lev[0];
  L.nfb = (L.F + S::FC - 1) / S::FC;
  L.fft_item0 = 0;
  const long long items = (long long)L.Jh * L.nfb;
  if (!group_takes(S::FC, L, ncu)) return -1;
  // 32-bit lane offsets within the rows of one group
  if ((double)S::FC * L.J * L.I * sizeof(T) >= 4294967296.0 || items > 0x7fffffff) return -1;
  a.nitems = (int)items;
  if constexpr (lds > 65536) {
    static const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_zonal_group<T, I, ANA>),
                                                    hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    (void)e;
  }
  constexpr int by_lds = (int)(most / lds), by_waves = S::WPE * 256 / S::NT;
  constexpr int per_cu = by_lds < by_waves ? by_lds : by_waves < 1 ? 1 : by_waves;
  const int nwg = ncu * per_cu < a.nitems ? ncu * per_cu : a.nitems;
  hipLaunchKernelGGL((k_zonal_group<T, I, ANA>), dim3(nwg), dim3(S::NT), lds, st, a);
  return (int)hipGetLastError();
}

}  // namespace

// Launch a's level; -1 if these kernels do not take it.
int SHT_GROUP_LAUNCH(const FftArgs1& a, int ncu, void* stream) {
  hipStream_t st = static_cast<hipStream_t>(stream);
  switch (a.lev[0].I) {
#define SHT_GROUP_CASE(i) \
  case i: return go<SHT_GROUP_T, i, SHT_GROUP_ANA>(a, ncu, st);
    SHT_GROUP_LENGTHS(SHT_GROUP_CASE)
#undef SHT_GROUP_CASE
    default: return -1;
  }
}

}  // namespace sht
