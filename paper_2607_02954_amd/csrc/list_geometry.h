// Geometry of the tile lists: which tiles a node reaches from where it is, and
// how (plain integer rules, also compiled for the host, where a test compares
// them with the cells that the kernels read).
#pragma once

#include "engine.h"

namespace mc {

static __host__ __device__ __forceinline__ int wrap_near(int v, int n) {   // v in [-n, 2n)
  return v < 0 ? v + n : (v >= n ? v - n : v);
}

// Class of home cell h (in [0, n)) for the tile [x0, x0 + tw) of a periodic
// axis: 0 own, 1 near, 2 far, 3 out of reach.
struct Reach {
  int near_, before, after;
  __host__ __device__ __forceinline__ explicit Reach(const WorldDev& w) {
    const bool mk = w.d_marker != nullptr;
    near_ = w.tl_near;
    before = far_reach_before(w.radius, mk);
    after = far_reach_after(w.radius, mk);
  }
  __host__ __device__ __forceinline__ int of_cell(int h, int x0, int tw, int n) const {
    if (h >= x0 && h < x0 + tw) return 0;
    const int a = h < x0 ? x0 - h : x0 - h + n;                  // cells before / after the tile (1 = next to it)
    const int b = h >= x0 + tw ? h - (x0 + tw - 1) : h - (x0 + tw - 1) + n;
    return a <= near_ || b <= near_ ? 1 : (a <= before || b <= after ? 2 : 3);
  }
};

// Neighbour q (0..7) of a tile: sides first (-x, +x, -y, +y), then corners.
static __host__ __device__ __forceinline__ constexpr int nb_dx(int q) { return q == 0 ? -1 : q == 1 ? 1 : q < 4 ? 0 : ((q & 1) ? 1 : -1); }
static __host__ __device__ __forceinline__ constexpr int nb_dy(int q) { return q < 2 ? 0 : q == 2 ? -1 : q == 3 ? 1 : (q < 6 ? -1 : 1); }
// Whether an axis of nt tiles has a neighbour in direction d of its own (two
// tiles are each other's neighbour once: in direction +1).
static __host__ __device__ __forceinline__ bool nb_exists(int d, int nt) { return d == 0 || nt >= 3 || (nt == 2 && d == 1); }
static __host__ __device__ __forceinline__ int nb_tile(int t, int d, int nt) { return wrap_near(t + d, nt); }

// f(tx, ty, class) for every tile that a node with home cell (hx, hy) reaches:
// the up to five tiles around its own per axis are tested (a reach of at most
// 11 cells spans a narrow last tile and the one beyond it).
template <int TILE, class F>
static __host__ __device__ __forceinline__ void for_reached_tiles(const WorldDev& w, int hx, int hy, F f) {
  constexpr int sh = tile_shift_of_side(TILE);
  const Reach R(w);
  const int cx = hx >> sh, cy = hy >> sh;
  const int nx = w.nx, ny = w.ny, ntx = w.ntx, nty = w.nty;
  const int mx = min(ntx, 5), my = min(nty, 5);
  for (int j = 0; j < my; ++j) {
    const int ty = nty <= 5 ? j : wrap_near(cy - 2 + j, nty);
    const int y0 = ty << sh, ky = R.of_cell(hy, y0, min(TILE, ny - y0), ny);
    if (ky > 2) continue;
    for (int i = 0; i < mx; ++i) {
      const int tx = ntx <= 5 ? i : wrap_near(cx - 2 + i, ntx);
      const int x0 = tx << sh, kx = R.of_cell(hx, x0, min(TILE, nx - x0), nx);
      if (kx <= 2) f(tx, ty, max(kx, ky));
    }
  }
}

// Whether tile (tx, ty) is (cx, cy) or one of its eight neighbours.
static __host__ __device__ __forceinline__ bool next_to(const WorldDev& w, int cx, int cy, int tx, int ty) {
  const int dx = abs(tx - cx), dy = abs(ty - cy);
  return (dx <= 1 || dx == w.ntx - 1) && (dy <= 1 || dy == w.nty - 1);
}

// How many tiles away along an axis of nt tiles of t cells (the last of `last`)
// a block can have integrated a node that reaches tile `at`: the reach and a
// small move are less than a tile, but not less than a narrow last one.
static __host__ __device__ __forceinline__ int axis_span(int at, int nt, int t, int last) {
  return last < t && (at == 0 || at == nt - 2) ? 2 : 1;
}

// Classes of a node with home (hx, hy) for the eight neighbours of tile
// (cx, cy), its home or the tile it just left, and whether it may reach a tile
// beyond them.
struct Classes {
  int kx, ky;                                    // for the tiles before, at and after, 2 bits each
  bool beyond;
  __host__ __device__ __forceinline__ int of(int q) const {
    return max((kx >> (2 * nb_dx(q) + 2)) & 3, (ky >> (2 * nb_dy(q) + 2)) & 3);
  }
};
// Classes along one axis of nt tiles of a node at place l of a tile of t cells
// (beside it by at most kSmallMove cells) that reaches no tile beyond its
// neighbours (Place).
static __host__ __device__ __forceinline__ int axis_classes(const Reach& R, int l, int t, int nt) {
  int k0 = l < 0 ? 0 : (l < R.near_ ? 1 : (l < R.after ? 2 : 3));
  int k1 = l < 0 ? (-l <= R.near_ ? 1 : 2) : (l >= t ? (l - t < R.near_ ? 1 : 2) : 0);
  int k2 = l >= t ? 0 : (t - l <= R.near_ ? 1 : (t - l <= R.before ? 2 : 3));
  if (nt < 3) {                                  // two tiles are neighbours on both sides
    k2 = nt == 2 ? min(k0, k2) : 3;
    k0 = 3;
    if (nt == 1) k1 = 0;
    else k1 = min(k1, 1);                        // (it may be nearer the other way round)
  }
  return k0 | (k1 << 2) | (k2 << 4);
}
// Place of home (hx, hy) relative to tile (cx, cy), the short way round, and
// whether it is one from which a node reaches no tile beyond the neighbours:
// at most kSmallMove cells beside the tile and, where a neighbour is the axis'
// narrow last tile, no nearer to it than the reach past it.  (Testing every
// tile around such nodes' own, as done for all nodes of a world with a narrow
// last tile before: 700 nodes on 72 x 50, 30.8 us per step; now 27.5.)
struct Place {
  int lx, ly;
  bool inside;
  static __host__ __device__ __forceinline__ bool fits(const Reach& R, int l, int t, int c, int nt, int last) {
    const int lo = nt > 2 && c == 0 ? max(-kSmallMove, R.after - last) : -kSmallMove;
    const int hi = t + (nt > 2 && c == nt - 2 ? min(kSmallMove, last - R.before) : kSmallMove);
    return l >= lo && l < hi;
  }
  __host__ __device__ __forceinline__ Place(const WorldDev& w, int side, int cx, int cy, int hx, int hy) {
    const Reach R(w);
    const int nx = w.nx, ny = w.ny, x0 = cx * side, y0 = cy * side, tw = min(side, nx - x0), th = min(side, ny - y0);
    lx = hx - x0;
    ly = hy - y0;
    lx += lx >= tw && 2 * lx > nx ? -nx : (lx < 0 && -2 * lx > nx ? nx : 0);
    ly += ly >= th && 2 * ly > ny ? -ny : (ly < 0 && -2 * ly > ny ? ny : 0);
    inside = fits(R, lx, tw, cx, w.ntx, nx - (w.ntx - 1) * side) && fits(R, ly, th, cy, w.nty, ny - (w.nty - 1) * side);
  }
};
template <int TILE>
static __host__ __device__ __forceinline__ Classes neighbour_classes(const WorldDev& w, int cx, int cy, int hx, int hy) {
  constexpr int sh = tile_shift_of_side(TILE);
  const Reach R(w);
  const int nx = w.nx, ny = w.ny, ntx = w.ntx, nty = w.nty;
  const Place p(w, TILE, cx, cy, hx, hy);
  Classes c;
  c.beyond = !p.inside;
  if (!c.beyond) {
    c.kx = axis_classes(R, p.lx, min(TILE, nx - cx * TILE), ntx);
    c.ky = axis_classes(R, p.ly, min(TILE, ny - cy * TILE), nty);
  } else {
    c.kx = c.ky = 0;
    for (int d = -1; d <= 1; ++d) {
      const int tx = nb_tile(cx, d, ntx) << sh, ty = nb_tile(cy, d, nty) << sh;
      c.kx |= (nb_exists(d, ntx) ? R.of_cell(hx, tx, min(TILE, nx - tx), nx) : 3) << (2 * d + 2);
      c.ky |= (nb_exists(d, nty) ? R.of_cell(hy, ty, min(TILE, ny - ty), ny) : 3) << (2 * d + 2);
    }
  }
  return c;
}

// What a node has to do with the neighbours along one axis: its class for the
// one that it reaches (2 bits), for the tile itself (2), which side that is,
// and whether it reaches both.
static __host__ __device__ __forceinline__ int axis_pairs(int classes) {
  const int k0 = classes & 3, k1 = (classes >> 2) & 3, k2 = classes >> 4;
  return min(k0, k2) | (k1 << 2) | (k0 < 3 ? 0 : 16) | (max(k0, k2) < 3 ? 32 : 0);
}
// The neighbours of a node that reaches at most one tile along each axis
// (more: it may reach others), as nearly all do: one beside it along x, one
// along y and the corner between them, with their classes.
struct Pairs {
  int dx, dy, side_x, side_y, corner;
  bool more;
  __host__ __device__ __forceinline__ Pairs(int x, int y, bool beyond) {
    const int kx = x & 3, ky = y & 3;
    more = beyond || ((x | y) & 32) != 0;
    dx = ((x >> 3) & 2) - 1;
    dy = ((y >> 3) & 2) - 1;
    side_x = max(kx, (y >> 2) & 3);
    side_y = max((x >> 2) & 3, ky);
    corner = max(kx, ky);
  }
  __host__ __device__ __forceinline__ explicit Pairs(const Classes& c) : Pairs(axis_pairs(c.kx), axis_pairs(c.ky), c.beyond) {}
  __host__ __device__ __forceinline__ int qx() const { return dx > 0; }
  __host__ __device__ __forceinline__ int qy() const { return 2 + (dy > 0); }
  __host__ __device__ __forceinline__ int qc() const { return 4 + (dx > 0) + 2 * (dy > 0); }
};

}  // namespace mc
