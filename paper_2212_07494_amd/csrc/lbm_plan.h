// Rules that choose a launch by sizes (host code without HIP): which kernel, which tiles.
#pragma once

#include <cstddef>
#include <cstdint>

namespace lbm {

// A launch holds fewer than 2^32 threads.
constexpr int64_t MAX_THREADS = int64_t(1) << 32;

// n / d rounded up, for n up to 2^31 - 1.
inline int ceil_div(int n, int d) { return n / d + (n % d != 0); }

// f(start, length) of the pieces of `size` that n < 2^31 is cut into (the last may be shorter).
template <class F>
void each_piece(int64_t n, int size, F f) {
  for (int64_t i = 0; i < n; i += size) f((int)i, (int)(n - i < size ? n - i : size));
}

// LDS bytes a workgroup may take for its data: what a compute unit has, and no more than one
// workgroup is allowed.
inline size_t workgroup_lds(int lds_cu, int lds_block) {
  const int least = lds_cu < lds_block ? lds_cu : lds_block;
  return least > 0 ? (size_t)least : 0;
}

// Whether a step's blocks take consecutive nodes of a layer, 128 a block: on ragged widths, where
// rows leave lanes idle, the block shape 64 x 3 stands for them (rows of 64 x 3 threads are no
// faster than 64 x 2 or 64 x 4 anywhere); every other shape is rows.  The tuner measures both
// kinds: D3Q27 of 72 columns FP32-shifted 27 us linear against 34 in rows, 150 columns FP64
// 111 / 128 tuned, but tuned 120 columns FP16-shifted 31.1 / 28.3, 160 columns FP32-shifted
// 61.7 / 58.6, and D2Q9 FP64 100000 x 2 9.4 / 6.4 (64 x 2: both rows in a block).
constexpr int LINEAR_SHAPE = 3, LINEAR_BY = 2;  // 64 x 3 stands for 128 threads
inline bool linear_blocks(int nx, int bx, int by) {
  return nx % 64 != 0 && bx == 64 && by == LINEAR_SHAPE;
}

// Launch of the single step before any tuning: block shape and variant (0 plain; on the
// scalar-base path 3 plain, 4 with non-temporal stores, 9 placed XCD by XCD).
//
// Blocks: rows of whole wavefronts, the widest among those that leave the fewest lanes idle (192
// columns: 64 x 4 rather than 128 x 2, D3Q27 FP64 516 against 631 us a step); consecutive nodes
// on ragged widths (D3Q27 FP64 300 x 100 x 100 222 against 383 us, 1000 x 64 x 64 300 / 352), but
// where rows stay the better (D3Q19 FP16-shifted 4097 x 16 x 16 21.8 linear / 20.1, D3Q39
// FP32-shifted 127^3 178 / 166, D2Q9 FP64 100000 x 2 9.4 / 6.4).  Few D2Q9 rows stand above one
// another, so that a compute unit reads its neighbours' rows once (FP64 256^2 64 x 4 4.3 against
// 256 x 1 5.6).
// Variant, by the bytes of the two population buffers: beyond the 256 MB last-level cache
// non-temporal stores (D3Q27 FP64 128^3 166 against 179 us; not where it is nearly full: D3Q19
// FP32-shifted 128 x 128 x 256 plain 52.5 / 54.5).  Within it XCD placement pays for consecutive
// nodes (D3Q19 FP32-shifted 100^3 26.3 against 32.1), on D2Q9 of a few rows an XCD (FP64 1024^2
// 22.9 / 24.6, but FP32-shifted 131072 x 4 10.1 / 7.7) and for rows (D3Q19 FP64 64^3 3%) but for
// those of binary16 (D3Q19 128^3 36.1 / 28.3), of D3Q27 (FP32-shifted 64 x 64 x 128 1.004 /
// 0.938 of plain rows) or with walls (D3Q19 FP32-shifted 64 x 128 x 64 walls y 14.8 / 14.1) well
// within the cache, with walls across x or solid nodes (D3Q19 FP32-shifted 128 x 128 x 96 5%)
// and the smallest (D2Q9 1000 x 1 3.2 / 2.9).  There the scalar-base path is the choice, which
// D3Q19 in FP32 does not earn (1-3% slower).
struct StepLaunch {
  int bx, by, variant;
};
inline StepLaunch default_launch(int Q, size_t elem, int nx, int ny, size_t bytes, bool across_x,
                                 bool walls) {
  constexpr size_t MIB = 1u << 20;
  StepLaunch l{};
  const int waves = ceil_div(nx, 64);
  const int64_t idle = ceil_div(nx, 256) * int64_t(256) - nx;  // lanes of rows of 256
  const bool rows = nx % 64 == 0 || (Q == 19 && elem == 2 && idle * 8 < nx) ||
                    (Q == 39 && nx < 256 && nx % 64 >= 62) || (Q == 9 && ny <= 2);
  if (!rows) {
    l.bx = 64;
    l.by = LINEAR_SHAPE;
  } else if (Q == 9 && ny > 1 && bytes <= 32 * MIB) {
    l.bx = 64;
    l.by = ny < 4 ? 2 : 4;
  } else {
    l.bx = waves % 4 == 0 ? 256 : waves % 2 == 0 ? 128 : 64;
    if (nx % 64 != 0 && nx > 256) l.bx = 256;
    l.by = 256 / l.bx;
  }
  const bool f32_q19 = elem == 4 && Q != 27;
  if (bytes > 320 * MIB)
    l.variant = 4;
  else if (bytes <= (Q == 9 ? 4 * MIB : MIB))
    l.variant = 3;
  else if (Q == 9)
    l.variant = ny >= 16 ? 9 : !rows || bytes <= 32 * MIB ? 3 : 0;
  else if (elem == 2 && rows)
    l.variant = 3;
  else if (bytes > 256 * MIB)
    l.variant = Q == 27 && rows ? 3 : 0;
  else if (!rows)
    l.variant = 9;
  else if (across_x)
    l.variant = f32_q19 ? 0 : 3;
  else if (bytes > 144 * MIB || (Q != 27 && !walls))
    l.variant = 9;
  else
    l.variant = f32_q19 ? 0 : 3;
  return l;
}

// Whether blocks of rows address through plane pointers where a pull may bounce back, rather
// than through 32-bit offsets (step_kernel's PLAIN).  across_x: walls across x or solid nodes,
// so that any block may bounce back; walls: walls across y or z, so that only blocks at them do.
// The offsets pay in binary16, and on D3Q27 where every block needs them (us a step, pointers /
// offsets: D3Q19 FP16-shifted 128^3 walls yz 34.8 / 31.1, D3Q27 FP64 128^3 walls xyz 168 / 162);
// elsewhere they cost more than they save (D3Q19 FP32-shifted 128 x 64 x 64 walls xyz 14.2 /
// 14.8, 256 x 128 x 128 walls y 102 / 105, D3Q27 FP64 96 x 96 x 128 walls y 90 / 91, D2Q9 FP64
// 1024^2 23.6 / 24.4).
inline bool rows_plain(int Q, size_t elem, bool across_x, bool walls) {
  if (elem == 2) return !across_x && !walls;
  return Q != 27 || !across_x;
}

// Several steps of a two-dimensional lattice in one launch (lbm_multistep.h): columns of a
// tile, steps of a launch (and of one on the smallest lattices), threads of a workgroup, and
// the most rows a plan lets a tile own.
constexpr int MULTI_W = 64;
constexpr int MULTI_STEPS = 5, MULTI_STEPS_MAX = 7;
constexpr int MULTI_THREADS = 512;
constexpr int MULTI_ROWS = 27;

// Launch of several steps in one pass over a two-dimensional lattice (lbm_multistep.h): K
// steps (odd, at least 3; 0: no such plan), tiles of ox x oy nodes in an ntx x nty grid,
// workgroups with `lds` bytes of LDS.
struct MultiPlan {
  int K, wx, ox, oy, ntx, nty;  // wx: columns of a wavefront's row (64 or 32)
  unsigned lds;
};

// The tiles a lattice's nx columns are split into, one beside the other, for K steps a
// launch: one of up to wx columns that wraps (or bounces) inside itself, else tiles that
// leave room for K - 1 columns more on each side.
inline int multi_columns(int nx, int K, int wx = MULTI_W) {
  const int room = nx <= wx ? nx : wx - 2 * (K - 1);
  return ceil_div(nx, room);
}
// LDS of a tile of oy rows, and the steps of a launch on a lattice of ny rows (0: none; a
// periodic lattice wraps once, and one of few rows would mostly compute its margins).
inline size_t multi_lds(int oy, int K, size_t elem, int wx = MULTI_W) {
  return (size_t)(oy + 2 * (K - 1)) * wx * 9 * elem;
}
inline int multi_steps(int ny, bool wy) { return wy || ny >= 12 ? MULTI_STEPS : (ny >= 3 ? 3 : 0); }
// Relative time of a launch of `tiles` tiles of oy rows: the compute units take them in
// turn, and a tile costs the rows of its K stages and about five more for its start and end.
// The fastest heights sit where the tiles just fill the compute units once, twice, ...:
// 512^2 FP32-shifted (10 columns) 22 rows, 240 tiles, 3.1 us a step against 4.4 at 20 rows,
// 260 tiles; 900^2 (17 columns) 20 rows, 765 tiles, 7.0 against 8.0 at 18 rows.  MULTI_ROWS
// keeps two workgroups a compute unit in FP32 (28 rows at 2048^2: 36 us a step, 27: 26).
inline double multi_cost(int64_t tiles, int oy, int K, int ncu) {
  return double((tiles + ncu - 1) / ncu) * (K * oy + K * (K - 1) + 5);
}

// Rows (wavefronts of 64 lanes) that the K stages of one column of tiles compute: tiles of oy
// rows down ny, each stage widened by up to K - 1 rows on both sides but not past a wall.
inline int64_t multi_rows(int ny, int oy, int K, bool wy) {
  const int64_t nty = ceil_div(ny, oy);
  auto tile = [&](int64_t y0) {
    const int64_t h = ny - y0 < oy ? ny - y0 : oy;
    int64_t rows = 0;
    for (int m = 0; m < K; ++m) {
      const int64_t below = wy && y0 < m ? y0 : m;
      const int64_t above = wy && ny - y0 - h < m ? ny - y0 - h : m;
      rows += below + h + above;
    }
    return rows;
  };
  if (nty <= 4) {
    int64_t rows = 0;
    for (int64_t t = 0; t < nty; ++t) rows += tile(t * oy);
    return rows;
  }
  return tile(0) + tile((nty - 1) * oy) + (nty - 2) * (K * (int64_t)oy + K * (K - 1));
}

// Whether launches of K steps are faster than single steps: a launch's tiles and their rows,
// which the compute units take in turn, against the nodes of a single step and its workgroups
// of 256 (which a batch's small domains leave mostly idle).  ns a tile, a row and a workgroup,
// us a launch, ps a node, for binary16, FP32 and FP64; fitted to 4,450 lattices and 250
// batches, where the choice is within 10% of the faster (us a step, single / several: 1 x 65535
// FP64 4.3 / 39, 12 x 65535 FP32-shifted 11.6 / 20.5, 2097152 x 1 walls y 24 / 44, but 2048 x
// 1024 24 / 13; 3000 domains of 3 x 200 FP64 41 / 384, of 16 x 16 18 / 38, but 732 of 64 x 64
// 74 / 42).
struct MultiRates {
  double tile, row, launch, block, node;
};
constexpr MultiRates LATTICE_RATES[3] = {
    {8.6, 0.48, 2.0, 0, 22}, {8.6, 0.48, 2.0, 0, 30}, {8.2, 0.75, 1.8, 0, 37}};
constexpr MultiRates BATCH_RATES[3] = {
    {9.4, 0.40, 4.0, 1.7, 8.2}, {9.4, 0.40, 4.0, 1.7, 8.2}, {12.5, 0.62, 2.8, 0.6, 25}};
inline bool multi_pays(const MultiRates (&rates)[3], size_t elem, int K, int64_t tiles,
                       int64_t rows, int64_t blocks, int64_t nodes, int ncu) {
  const MultiRates &r = rates[elem == 2 ? 0 : elem == 4 ? 1 : 2];
  const double turns = double((tiles + ncu - 1) / ncu) * ncu / double(tiles);
  const double several = turns * (double(tiles) * r.tile + double(rows) * r.row) / K * 1e-3;
  return several < r.launch + double(blocks) * r.block * 1e-3 + double(nodes) * r.node * 1e-6;
}

// Steps, columns and rows of the tiles.  A launch whose tiles each find a compute unit of
// their own lasts as long as one tile, whose stages take their rows in passes of the
// workgroup's wavefronts: about six rows' worth of latency a pass besides the rows themselves,
// after 22 for the launch.  There rows of 32 columns, two to a wavefront, halve the passes, and
// the idle units pay for the wider margins (us a step, five steps on 64 columns, on 32, seven
// on 32: 64 x 32 BGK FP64 1.83 / 1.62 / 1.57, 50 x 200 SMRT FP64 1.63 / 1.50 / 1.46, 128^2 FP64
// 1.60 / 1.49 / 1.42, 256^2 FP64 2.09 / 1.94 / 2.00); and more steps a launch, where their rows
// still make one pass.  Launches with more tiles than units are bound by the rows (multi_cost),
// if they pay at all (multi_pays).
inline MultiPlan multi_plan(int nx, int ny, bool wy, size_t elem, size_t lds, int ncu) {
  MultiPlan p{};
  // a plane's byte offsets are 32-bit in the kernel
  if (ncu < 1 || (uint64_t)nx * ny * elem >= (1ull << 32)) return p;
  constexpr int WAVES = MULTI_THREADS / 64;
  const int few = multi_steps(ny, wy);
  double best = 0;
  auto consider = [&](int K, int wx, bool single) {
    const int rpw = 64 / wx, ntx = multi_columns(nx, K, wx);
    for (int oy = 1; oy <= MULTI_ROWS && multi_lds(oy, K, elem, wx) <= lds; ++oy) {
      const int nty = ceil_div(ny, oy);
      const int64_t tiles = (int64_t)ntx * nty;
      if (single != (tiles <= ncu) || tiles * MULTI_THREADS >= MAX_THREADS) continue;
      double cost = multi_cost(tiles, oy, K, ncu);
      if (single) {
        cost = 22;
        for (int s = 0; s < K; ++s) {
          const int rows = (oy + 2 * s + rpw - 1) / rpw;  // of the last stage first
          cost += 6 * ((rows + WAVES - 1) / WAVES) + rows;
        }
        cost /= K;
      }
      if (p.K && cost >= best) continue;
      best = cost;
      p.K = K;
      p.wx = wx;
      p.ntx = ntx;
      p.oy = oy;
      p.nty = nty;
    }
  };
  if (few) {
    consider(few, MULTI_W, true);
    consider(few, 32, true);
    if (wy || ny >= 2 * MULTI_STEPS_MAX) consider(MULTI_STEPS_MAX, 32, true);
    if (!p.K) {
      consider(few, MULTI_W, false);
      if (p.K && !multi_pays(LATTICE_RATES, elem, p.K, (int64_t)p.ntx * p.nty,
                             p.ntx * multi_rows(ny, p.oy, p.K, wy), 0, (int64_t)nx * ny, ncu))
        return MultiPlan{};
    }
  }
  if (!p.K) return p;
  p.ox = ceil_div(nx, p.ntx);
  p.lds = (unsigned)multi_lds(p.oy, p.K, elem, p.wx);
  return p;
}

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
  if (waves_blocks(nx, rows) * WV_THREADS >= MAX_THREADS) return true;
  const double chunk = 25.0 * Q + 2.0 * Q * t.ngroups + 2.0 * t.nwaves + 8.0 * t.longest;
  return (nx + WV_X - 1) / WV_X * chunk > 1.3 * nx * t.nwaves;
}

// Workgroups of 256 threads of a batch's single steps, which walk its tiles: blocks_per_cu a
// compute unit, or (0) one a tile (a multiple of the XCD count, so that the XCD-contiguous walk
// applies) as far as a launch goes.
inline int batch_grid(int blocks_per_cu, int ncu, int ntiles) {
  if (blocks_per_cu) return blocks_per_cu * ncu;
  const int64_t most = MAX_THREADS / 256 - 8, grid = ((int64_t)ntiles + 7) / 8 * 8;
  return (int)(grid < most ? grid : most);
}

}  // namespace lbm
