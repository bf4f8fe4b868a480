// Group kernels of the zonal analysis, FP32.
#define SHT_GROUP_T float
#define SHT_GROUP_ANA true
#define SHT_GROUP_LAUNCH launch_zonal_group_analysis_f32
#include "sht_zonal_group_impl.h"
