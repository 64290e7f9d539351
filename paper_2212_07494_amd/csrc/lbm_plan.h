// Rules that choose a launch by sizes (host code without HIP): which kernel, which tiles.
#pragma once

#include <cstdint>

namespace lbm {

// Fourier waves for waves_kernel (device arrays), sorted into groups of one k_x: group g's
// waves are [group_start[g], group_start[g + 1]), `longest` of them at most, and its wavenumber
// group_k[g]; per wave k_x, k_y, k_z and 0 (k) and the Q amplitudes' (re, im) pairs, times
// e^{i phase}.  Wavenumbers are reduced to [0, n_a).
struct WaveTable {
  int nwaves, ngroups, longest;
  const int *group_start, *group_k, *k;
  const double *amp;
};

// waves_kernel's workgroups: WV_ROWS rows of WV_X nodes each.
constexpr int WV_ROWS = 4, WV_X = 128, WV_THREADS = 256;
inline int64_t waves_blocks(int nx, int64_t rows) {
  return (rows + WV_ROWS - 1) / WV_ROWS * ((nx + WV_X - 1) / WV_X);
}

// Whether a node sums its own waves (waves_node_kernel) rather than its row's (waves_kernel).
// In units of about 4 ps, WV_X nodes of a row cost 25 Q and 2 Q a group for their own sums, 2 a
// wave for its factor and 8 a wave of the longest group, whose Q amplitudes are summed by as
// many threads; a node's own sum costs 1.3 a wave.  So rows of few nodes and few waves are
// cheaper by node (us a start, by row / by node, D3Q27 FP64 of 2 million nodes: 3 columns 185
// waves 7985 / 1864; 8 columns 4 waves 661 / 103; 32 columns 185 waves 853 / 1869, 20 waves
// 462 / 261; 128 columns 20 waves 180 / 270, 4 waves 140 / 104).
inline bool waves_by_node(const WaveTable &t, int Q, int nx, int64_t rows) {
  if (waves_blocks(nx, rows) * WV_THREADS >= (int64_t(1) << 32)) return true;
  const double chunk = 25.0 * Q + 2.0 * Q * t.ngroups + 2.0 * t.nwaves + 8.0 * t.longest;
  return (nx + WV_X - 1) / WV_X * chunk > 1.3 * nx * t.nwaves;
}

}  // namespace lbm
