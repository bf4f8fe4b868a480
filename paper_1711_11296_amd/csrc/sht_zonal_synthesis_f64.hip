// Group kernels of the zonal synthesis, FP64.
#define SHT_GROUP_T double
#define SHT_GROUP_ANA false
#define SHT_GROUP_LAUNCH launch_zonal_group_synthesis_f64
#include "sht_zonal_group_impl.h"
