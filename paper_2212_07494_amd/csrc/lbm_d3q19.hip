// Kernels of the D3Q19 lattice (see lbm_lattice_impl.h).
#define LBM_LAT D3Q19
#define LBM_OPS ops_d3q19
#define LBM_MULTI nullptr
#define LBM_BATCH_MULTI nullptr
#include "lbm_lattice_impl.h"
