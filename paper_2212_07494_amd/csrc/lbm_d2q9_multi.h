// Launchers of the D2Q9 multi-step kernels (lbm_multistep.h); included by lbm_d2q9.hip only.
#pragma once
#include "lbm_multistep.h"

namespace lbm {
namespace {

template <class S, class T, int COLL>
hipError_t launch(const LaunchDesc &d, const MultiPlan &p, int k, const double *gs,
                  hipStream_t s) {
  MultiDom<T> D;
  D.fin = d.fin;
  D.fout = d.fout;
  D.nx = d.geo.nx;
  D.ny = d.geo.ny;
  D.ps = d.geo.ps;
  D.wx = d.geo.wall[0];
  D.wy = d.geo.wall[1];
  D.smask = d.geo.smask;
  D.tab = static_cast<const T *>(d.gtab);
  D.axis = d.gk ? 3 : d.g_axis;
  D.n = d.gk ? d.geo.N : d.g_n;
  D.shift = T(d.shift);
  D.c0 = T(d.c0);
  D.c1 = T(d.c1);
  D.c2 = T(d.c2);
  D.c3 = T(d.c3);
  D.c4 = T(d.c4);
  MultiScale<T> sc;
  for (int j = 0; j < MULTI_STEPS_MAX; ++j) sc.v[j] = T(gs && j < k ? gs[j] : d.gscale);
  sc.sdev = d.gs_dev;
  sc.sctr = d.gs_ctr;
  sc.sj = d.gs_j;
  const dim3 grid(p.ntx * p.nty), block(MULTI_THREADS);
  const auto kernel = p.wx == 32 ? (d.gk ? multi_step_kernel<D2Q9, COLL, S, T, 32, true>
                                         : multi_step_kernel<D2Q9, COLL, S, T, 32, false>)
                                 : (d.gk ? multi_step_kernel<D2Q9, COLL, S, T, 64, true>
                                         : multi_step_kernel<D2Q9, COLL, S, T, 64, false>);
  hipLaunchKernelGGL(kernel, grid, block, p.lds, s, D, sc, k, p.ox, p.oy, p.ntx);
  return hipGetLastError();
}

template <class S, class T>
hipError_t by_collision(const LaunchDesc &d, const MultiPlan &p, int k, const double *gs,
                        hipStream_t s) {
  switch (d.coll) {
    case 0: return launch<S, T, 0>(d, p, k, gs, s);
    case 1: return launch<S, T, 1>(d, p, k, gs, s);
    case 2: return launch<S, T, 2>(d, p, k, gs, s);
    case 4: return launch<S, T, 4>(d, p, k, gs, s);
    case 5: return launch<S, T, 5>(d, p, k, gs, s);
    case 7: return launch<S, T, 7>(d, p, k, gs, s);
    default: return hipErrorInvalidValue;
  }
}

template <class S, class T, int COLL>
hipError_t launch_batch(const BatchLaunch &b, int k, hipStream_t s) {
  hipLaunchKernelGGL((batch_multi_kernel<D2Q9, COLL, S, T>), dim3(b.nmulti), dim3(MULTI_THREADS),
                     b.multi_lds, s, static_cast<const S *>(b.fin), static_cast<S *>(b.fout),
                     static_cast<const T *>(b.gbuf), static_cast<const BatchDom *>(b.doms),
                     static_cast<const BatchMultiTile *>(b.multi), b.active, T(b.shift), k);
  return hipGetLastError();
}

template <class S, class T>
hipError_t by_collision(const BatchLaunch &b, int k, hipStream_t s) {
  return b.coll == 0 ? launch_batch<S, T, 0>(b, k, s) : launch_batch<S, T, 1>(b, k, s);
}

}  // namespace

hipError_t multi_step_d2q9(const LaunchDesc &d, const MultiPlan &p, int k, const double *gs,
                           hipStream_t s) {
  if (k < 3 || k > p.K || k % 2 == 0) return hipErrorInvalidValue;
  switch (d.storage) {
    case 0: return by_collision<double, double>(d, p, k, gs, s);
    case 1:
    case 2: return by_collision<float, float>(d, p, k, gs, s);
    case 3: return by_collision<_Float16, float>(d, p, k, gs, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t batch_multi_d2q9(const BatchLaunch &b, int k, hipStream_t s) {
  if (k < 3 || k > MULTI_STEPS || k % 2 == 0 || b.nmulti < 1) return hipErrorInvalidValue;
  switch (b.storage) {
    case 0: return by_collision<double, double>(b, k, s);
    case 1:
    case 2: return by_collision<float, float>(b, k, s);
    case 3: return by_collision<_Float16, float>(b, k, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace lbm
