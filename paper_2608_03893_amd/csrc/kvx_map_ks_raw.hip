// The kernels of kvx_map_ks.hip for maps read as given.
#define KVX_RAW_MAPS 1
#include "kvx_map_ks.hip"
