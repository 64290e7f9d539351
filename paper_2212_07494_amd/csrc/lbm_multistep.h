// Several steps of a two-dimensional lattice in one launch (gfx950).
//
// A workgroup owns a tile of ox x oy nodes and takes it K steps ahead.  Stage s = 0 .. K-1
// computes the step's post-collision populations on the tile widened by K-1-s nodes on each
// side, so the last stage needs nothing from another workgroup: stage 0 pulls from the
// populations in memory, the stages between exchange theirs through LDS, and the last stage
// writes the tile back.  Every node value is the one the single-step kernel computes, in the
// same operations; the nodes of the widened tile are computed more than once.
//
// Layout.  A wavefront works on one row of up to WX = 64 nodes, x = x0 - hx + lane; the rows of
// a stage are dealt to the workgroup's wavefronts in turn.  Row and plane addresses are then
// uniform (scalar), and a lane holds three column offsets (its own and its neighbours') for
// the whole launch.  A lattice of at most WX columns is one tile wide and wraps (or bounces)
// inside it: no widening in x.  LDS holds slot (row, i, x) at (row Q + i) WX + x, so all of a
// node's slots are at constant distances from its own and a row of lanes is free of bank
// conflicts.  WX = 32 puts two rows into a wavefront (multi_plan says when).
//
// One copy of the populations in LDS is enough.  Slot (i, y) in the kernel's usual meaning
// ("own": the post-collision population i of node y) is read by node y + e_i alone.  A node
// that has pulled its populations from the slots (i, x - e_i) puts its new population opp(i)
// back into the very slot (i, x - e_i) it read (it travels to x - e_i); in that meaning
// ("swapped") the next stage's node finds population i in its own slot opp(i), and writes its
// results to its own slots, in the usual meaning again.  Every stage's reads and writes of a
// node are the same set of slots, no two nodes share one, and one barrier a stage suffices.
// Halfway bounce-back is the pull from the own slot opp(i), which no other node reads (its
// reader would lie beyond the wall); in the swapped meaning it needs no case of its own.
//
// What bounds it.  A step of its own reads and writes every population in memory and pays a
// launch; on the lattices that fit the caches the launch and the latency of its loads are all
// there is to a step (3 us at 64 x 32).  Five steps a launch share one launch and one pass
// over memory, and the vector ALU becomes the bound: about 240 instructions a node and stage,
// twice the bare arithmetic of the widened tile's nodes.  With one or two wavefronts a SIMD,
// as on the smallest lattices, an instruction takes about eight cycles instead of four, and a
// stage's chain of them (1,400 to 2,500 cycles) is the floor.  Measured, us per step, single
// steps against these launches as planned (SMRT but for the first, in one run): 64 x 32 BGK
// FP64 3.0 / 1.57; 50 x 200 FP64 3.0 / 1.45; 512^2 FP64 10.0 / 4.3; 1024^2 FP32-shifted 13.8 /
// 7.9, FP64 25.3 / 14.0; 2048^2 FP32-shifted 57 / 26; a batch of 512 domains (5.8 million
// nodes) FP32-shifted 120 / 49.  A launch of that batch reads its populations once (0.21 GB) and
// writes 1.8 times them (0.38 GB, by the counters).
//
// Why five.  Fewer leave more of the launch, more widen the tile; three, five and seven steps
// on 64-column tiles, us per step: 128^2 FP64 1.76 / 1.60 / 1.69, 512^2 FP32-shifted 3.10 / 2.91 /
// 2.80, 900^2 6.5 / 6.8 / 6.9, 1024^2 8.8 / 8.0 / 9.4, FP64 15.1 / 13.8 / 15.5, 2048^2
// FP32-shifted 30 / 26 / 37.  Seven pay on 32-column tiles while their rows make one pass of the
// wavefronts (32^2 FP64 1.27 against 1.35).  512 threads: more wavefronts than a stage has rows
// idle, and two workgroups of eight wavefronts hide each other's barriers (1024 threads: 10.3
// against 8.1 at 1024^2).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "lbm_batch_kernels.h"
#include "lbm_internal.h"
#include "lbm_kernels.h"

namespace lbm {

// What a tile's K steps need to know of its lattice.
template <class T>
struct MultiDom {
  const void *fin;
  void *fout;
  int nx, ny;
  int64_t ps;            // plane stride
  int wx, wy;            // walls across x, y
  const uint32_t *smask; // solid mask words, or NULL
  const T *tab;          // force table
  int axis, n;           // as ForceRef; axis 3: a full field of n nodes a plane
  T shift, c0, c1, c2, c3, c4;
};

// The tile: its first owned node and its owned size.
struct MultiTile {
  int x0, y0, ox, oy;
};

// Force factors of the launch's steps: one value, or from device memory (graph replays).
template <class T>
struct MultiScale {
  T v[MULTI_STEPS_MAX];
  const double *sdev;  // sdev[*sctr + sj + s] if set
  const int64_t *sctr;
  int sj;
};

// LDS pointers in their own address space (a pointer of either space would make every access
// a flat one).
template <class S>
using LdsPtr = __attribute__((address_space(3))) S *;

// The tile widened by H = K - 1 (no further than a wall), and a lane's columns.
struct MultiFrame {
  int hx, hy, ex, ey;  // margins below the owned nodes, extents
  int gx, gl, gr;      // this lane's lattice column and its neighbours'
  int col, cl, cr;     // its and the neighbours' columns in the tile
  bool at_l, at_r;     // a wall beside this column
  int wave, nwaves, lane;
  int sub;             // its row among the wavefront's
};

template <int WX, class T>
__device__ __forceinline__ MultiFrame multi_frame(const MultiDom<T> &D, const MultiTile &tile,
                                                  int H) {
  MultiFrame f;
  f.lane = threadIdx.x & 63;
  f.col = f.lane % WX;
  f.sub = f.lane / WX;
  f.wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  f.nwaves = blockDim.x >> 6;
  const bool whole = D.nx <= WX;  // one tile wide: wraps or bounces inside the tile
  const int room_l = D.wx ? min(H, tile.x0) : H;
  const int room_r = D.wx ? min(H, D.nx - tile.x0 - tile.ox) : H;
  f.hx = whole ? 0 : room_l;
  f.ex = f.hx + tile.ox + (whole ? 0 : room_r);
  f.hy = D.wy ? min(H, tile.y0) : H;
  f.ey = f.hy + tile.oy + (D.wy ? min(H, D.ny - tile.y0 - tile.oy) : H);
  int gx = tile.x0 - f.hx + f.col;
  gx = gx < 0 ? gx + D.nx : (gx >= D.nx ? gx - D.nx : gx);
  f.gx = gx;
  f.gl = gx == 0 ? D.nx - 1 : gx - 1;
  f.gr = gx == D.nx - 1 ? 0 : gx + 1;
  f.cl = whole && f.col == 0 ? D.nx - 1 : f.col - 1;
  f.cr = whole && f.col == D.nx - 1 ? 0 : f.col + 1;
  f.at_l = D.wx && gx == 0;
  f.at_r = D.wx && gx == D.nx - 1;
  return f;
}

// A wavefront's value of lane src (uniform).
__device__ __forceinline__ float lane_value(float v, int src) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), src));
}
__device__ __forceinline__ double lane_value(double v, int src) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), src),
                          __builtin_amdgcn_readlane(__double2loint(v), src));
}

// The force and its factors, loaded once a launch (each stage would wait for them again):
// a table along y by the row in the tile (lane r holds row r), any other table by this
// lane's column, the factors by the stage (lane s holds stage s).  A full field is read by
// each stage.
template <class T>
struct MultiForce {
  T lane[2], factor;
  bool by_row;
};

template <class T>
__device__ __forceinline__ MultiForce<T> multi_force(const MultiDom<T> &D, const MultiTile &tile,
                                                     const MultiFrame &f,
                                                     const MultiScale<T> &scale, int K) {
  MultiForce<T> F;
  F.by_row = D.axis == 1;
  int gy = tile.y0 - f.hy + min(f.lane, f.ey - 1);
  gy = gy < 0 ? gy + D.ny : (gy >= D.ny ? gy - D.ny : gy);
  const int c = D.axis == 0 ? min(f.gx, D.nx - 1) : (D.axis == 1 ? gy : 0);
  for (int a = 0; a < 2; ++a) F.lane[a] = D.axis == 3 ? T(0) : D.tab[a * D.n + c];
  const int s = min(f.lane, K - 1);
  F.factor = scale.sdev ? T(scale.sdev[*scale.sctr + scale.sj + s]) : scale.v[s];
  return F;
}

// Where a stage's populations come from and go to: from memory into the own slots; from the
// own slots into the swapped ones; back; from the swapped slots to memory.
enum { ST_FIRST = 0, ST_PULL = 1, ST_SWAP = 2, ST_LAST = 3 };

// Stage s of the tile.  BOUNCE: some node of the widened tile may bounce back (walls or
// solid nodes).
template <class L, int COLL, class S, class T, int WX, bool BOUNCE, bool FIELD, int STAGE>
__device__ __forceinline__ void multi_stage(const MultiDom<T> &D, const MultiTile &tile,
                                            const MultiFrame &f, const MultiForce<T> &F, int m,
                                            T sc, LdsPtr<S> lds) {
  static_assert(L::D == 2);
  constexpr int Q = L::Q;
  constexpr int ROW = Q * WX;    // LDS elements of a row
  constexpr int RPW = 64 / WX;   // rows of a wavefront
  const S *__restrict__ fin = static_cast<const S *>(D.fin);
  S *__restrict__ fout = static_cast<S *>(D.fout);
  const int nx = D.nx, ny = D.ny;
  const int xlo = max(0, f.hx - m), xhi = min(f.ex, f.hx + tile.ox + m);
  const int ylo = max(0, f.hy - m), yhi = min(f.ey, f.hy + tile.oy + m);
  const bool in_x = f.col >= xlo && f.col < xhi;
  for (int rb = ylo + f.wave * RPW; rb < yhi; rb += f.nwaves * RPW) {
    const int r = RPW == 1 ? rb : rb + f.sub;  // uniform where a wavefront has one row
    const bool live = in_x && (RPW == 1 || r < yhi);
    int gy = tile.y0 - f.hy + r;
    gy = gy < 0 ? gy + ny : (gy >= ny ? gy - ny : gy);
    const int row = gy * nx;
    T g[3] = {F.lane[0], F.lane[1], T(0)};
    if (!FIELD && F.by_row)  // with every lane of the wavefront active
      for (int a = 0; a < 2; ++a)
        g[a] = RPW == 1 ? lane_value(F.lane[a], r) : __shfl(F.lane[a], r, 64);
    if (!live) continue;
    uint32_t sm = 0;
    if constexpr (BOUNCE) {
      if (D.smask) sm = D.smask[row + f.gx];
      if (sm & SOLID_NODE) continue;
    }
    // whether population i bounces back into this node (its source is across a wall or
    // solid)
    const bool at_b = BOUNCE && D.wy && gy == 0, at_t = BOUNCE && D.wy && gy == ny - 1;
    auto bounces = [&](auto I) -> bool {
      constexpr int i = decltype(I)::value;
      bool b = (sm >> i) & 1u;
      if constexpr (L::E[i][0] > 0) b |= f.at_l;
      if constexpr (L::E[i][0] < 0) b |= f.at_r;
      if constexpr (L::E[i][1] > 0) b |= at_b;
      if constexpr (L::E[i][1] < 0) b |= at_t;
      return b;
    };
    if (FIELD)
      for (int a = 0; a < 2; ++a) g[a] = *at_offset(D.tab + ((int64_t)a * D.n + row), f.gx);
    for (int a = 0; a < 2; ++a) g[a] = g[a] * sc;
    const LdsPtr<S> lrow = lds + r * ROW;
    const LdsPtr<S> own = lrow + f.col, left = lrow + f.cl, right = lrow + f.cr;
    // the slot population i is pulled from
    auto source = [&](auto I) -> LdsPtr<S> {
      constexpr int i = decltype(I)::value;
      constexpr int ex = L::E[i][0], ey = L::E[i][1];
      LdsPtr<S> p = (ex > 0 ? left : (ex < 0 ? right : own)) + (i * WX - ey * ROW);
      if constexpr (BOUNCE && i > 0)
        if (bounces(I)) p = own + L::OPP[i] * WX;
      return p;
    };
    T d[Q];
    if constexpr (STAGE == ST_FIRST) {
      const int rowb = gy == 0 ? (ny - 1) * nx : row - nx;
      const int rowt = gy == ny - 1 ? 0 : row + nx;
      static_for<Q>([&](auto I) {
        constexpr int i = decltype(I)::value;
        constexpr int ex = L::E[i][0], ey = L::E[i][1];
        const S *plane = fin + i * D.ps;
        uint32_t o = (uint32_t)((ey > 0 ? rowb : (ey < 0 ? rowt : row)) +
                                (ex > 0 ? f.gl : (ex < 0 ? f.gr : f.gx)));
        if constexpr (BOUNCE && i > 0) {
          const bool b = bounces(I);
          const S *p = b ? fin + L::OPP[i] * D.ps : plane;
          d[i] = T(*at_offset(p, b ? (uint32_t)(row + f.gx) : o));
        } else {
          d[i] = T(*at_offset(plane, o));
        }
      });
    } else if constexpr (STAGE == ST_PULL) {
      static_for<Q>([&](auto I) { d[decltype(I)::value] = T(*source(I)); });
    } else {
      static_for<Q>([&](auto I) {
        constexpr int i = decltype(I)::value;
        d[i] = T(own[L::OPP[i] * WX]);
      });
    }
    collide_node<L, COLL>(d, D.shift, g, D.c0, D.c1, D.c2, D.c3, D.c4);
    if constexpr (STAGE == ST_LAST) {
      static_for<Q>([&](auto I) {
        constexpr int i = decltype(I)::value;
        *at_offset(fout + i * D.ps, (uint32_t)(row + f.gx)) = S(d[i]);
      });
    } else if constexpr (STAGE == ST_PULL) {
      static_for<Q>([&](auto I) { *source(I) = S(d[L::OPP[decltype(I)::value]]); });
    } else {
      static_for<Q>([&](auto I) {
        constexpr int i = decltype(I)::value;
        own[i * WX] = S(d[i]);
      });
    }
  }
}

// K steps of a tile (K odd, >= 3: the last stage then reads the swapped slots).
template <class L, int COLL, class S, class T, int WX, bool BOUNCE, bool FIELD>
__device__ __forceinline__ void multi_tile(const MultiDom<T> &D, const MultiTile &tile, int K,
                                           const MultiScale<T> &scale, LdsPtr<S> lds) {
  const int H = K - 1;
  const MultiFrame f = multi_frame<WX>(D, tile, H);
  const MultiForce<T> F = multi_force(D, tile, f, scale, K);
  auto factor = [&](int s) -> T { return lane_value(F.factor, s); };
  multi_stage<L, COLL, S, T, WX, BOUNCE, FIELD, ST_FIRST>(D, tile, f, F, H, factor(0), lds);
  __syncthreads();
  for (int s = 1;; s += 2) {
    multi_stage<L, COLL, S, T, WX, BOUNCE, FIELD, ST_PULL>(D, tile, f, F, H - s, factor(s), lds);
    __syncthreads();
    if (s + 1 == H) break;
    multi_stage<L, COLL, S, T, WX, BOUNCE, FIELD, ST_SWAP>(D, tile, f, F, H - s - 1, factor(s + 1), lds);
    __syncthreads();
  }
  multi_stage<L, COLL, S, T, WX, BOUNCE, FIELD, ST_LAST>(D, tile, f, F, 0, factor(H), lds);
}

// Tile t with or without bounce-back, whichever its widened nodes need.
template <class L, int COLL, class S, class T, int WX, bool FIELD>
__device__ __forceinline__ void multi_run(const MultiDom<T> &D, const MultiTile &t, int K,
                                          const MultiScale<T> &scale, unsigned char *lds_raw) {
  const bool bounce = D.smask || (D.wx && (t.x0 < K || t.x0 + t.ox > D.nx - K)) ||
                      (D.wy && (t.y0 < K || t.y0 + t.oy > D.ny - K));
  const LdsPtr<S> lds = (LdsPtr<S>)(lds_raw);
  if (bounce)
    multi_tile<L, COLL, S, T, WX, true, FIELD>(D, t, K, scale, lds);
  else
    multi_tile<L, COLL, S, T, WX, false, FIELD>(D, t, K, scale, lds);
}

template <class L, int COLL, class S, class T, int WX, bool FIELD>
__global__ void __launch_bounds__(MULTI_THREADS)
    multi_step_kernel(MultiDom<T> D, MultiScale<T> scale, int K, int ox, int oy, int ntx) {
  extern __shared__ __align__(16) unsigned char multi_lds_raw[];
  const int b = (int)xcd_block(blockIdx.x, gridDim.x);
  const int ty = b / ntx, tx = b - ty * ntx;
  MultiTile t;
  t.x0 = tx * ox;
  t.y0 = ty * oy;
  t.ox = min(ox, D.nx - t.x0);
  t.oy = min(oy, D.ny - t.y0);
  multi_run<L, COLL, S, T, WX, FIELD>(D, t, K, scale, multi_lds_raw);
}

// The same over the tiles of a batch: one workgroup a tile, none for inactive domains.
template <class L, int COLL, class S, class T>
__global__ void __launch_bounds__(MULTI_THREADS)
    batch_multi_kernel(const S *__restrict__ fin, S *__restrict__ fout,
                       const T *__restrict__ gbuf, const BatchDom *__restrict__ doms,
                       const BatchMultiTile *__restrict__ tiles, const int *__restrict__ active,
                       T shift, int K) {
  extern __shared__ __align__(16) unsigned char multi_lds_raw[];
  const BatchMultiTile bt = tiles[xcd_block(blockIdx.x, gridDim.x)];
  if (!active[bt.dom]) return;
  const BatchDom &dm = doms[bt.dom];
  MultiDom<T> D;
  D.fin = fin + dm.base;
  D.fout = fout + dm.base;
  D.nx = dm.nx;
  D.ny = dm.ny;
  D.ps = dm.ps;
  D.wx = dm.wall[0];
  D.wy = dm.wall[1];
  D.smask = nullptr;
  D.tab = gbuf + dm.goff;
  D.axis = dm.gaxis;
  D.n = dm.gn;
  D.shift = shift;
  D.c0 = T(dm.c0);
  D.c1 = T(dm.c1);
  D.c2 = D.c3 = D.c4 = T(0);
  MultiScale<T> one{};
  for (int s = 0; s < MULTI_STEPS_MAX; ++s) one.v[s] = T(1);
  const MultiTile t = {bt.x0, bt.y0, bt.ox, bt.oy};
  if (dm.gaxis == 3)
    multi_run<L, COLL, S, T, MULTI_W, true>(D, t, K, one, multi_lds_raw);
  else
    multi_run<L, COLL, S, T, MULTI_W, false>(D, t, K, one, multi_lds_raw);
}

}  // namespace lbm
