// Group kernels of the zonal analysis, FP64.
#define SHT_GROUP_T double
#define SHT_GROUP_ANA true
#define SHT_GROUP_LAUNCH launch_zonal_group_analysis_f64
#include "sht_zonal_group_impl.h"
