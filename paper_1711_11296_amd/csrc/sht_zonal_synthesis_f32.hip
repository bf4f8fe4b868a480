// Group kernels of the zonal synthesis, FP32.
#define SHT_GROUP_T float
#define SHT_GROUP_ANA false
#define SHT_GROUP_LAUNCH launch_zonal_group_synthesis_f32
#include "sht_zonal_group_impl.h"
