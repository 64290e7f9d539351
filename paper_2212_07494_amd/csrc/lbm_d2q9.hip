// Kernels of the D2Q9 lattice (see lbm_lattice_impl.h).
#define LBM_LAT D2Q9
#define LBM_OPS ops_d2q9
#define LBM_MULTI &multi_step_d2q9
#define LBM_BATCH_MULTI &batch_multi_d2q9
#include "lbm_lattice_impl.h"
#include "lbm_d2q9_multi.h"
