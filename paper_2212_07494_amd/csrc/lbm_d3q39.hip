// Kernels of the D3Q39 lattice (see lbm_lattice_impl.h).
#define LBM_LAT D3Q39
#define LBM_OPS ops_d3q39
#define LBM_MULTI nullptr
#define LBM_BATCH_MULTI nullptr
#include "lbm_lattice_impl.h"
