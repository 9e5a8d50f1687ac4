// Brute-force check of the tile lists' geometry (list_geometry.h) on the host:
// prints the number of checks made, or the first that fails.
#include <cstdio>
#include <cstdlib>
#include <set>
#include <vector>

#include "list_geometry.h"

using namespace mc;

static long n_checks = 0;
static char where[256];
#define CHECK(cond)                                                     \
  do {                                                                  \
    ++n_checks;                                                         \
    if (!(cond)) {                                                      \
      std::printf("line %d: %s fails at %s\n", __LINE__, #cond, where); \
      std::exit(1);                                                     \
    }                                                                   \
  } while (0)

// The class that the kernels' reads ask for, from the cells alone.  A node of
// home h has weights on cells h - 1 .. h + 2, its two-layer markers (home moved
// by at most one cell) on h - 2 .. h + 3.  The spread needs the tile's cells, in
// the one-kernel step those that its own nodes (their markers) interpolate from;
// the filter needs the tile, the ring of its differences and R cells of support.
struct Axis {
  int n, t, nt, R;
  bool mk, fused;
  int first(int c) const { return c * t; }
  int width(int c) const { return c == nt - 1 ? n - c * t : t; }
  int tile_of(int h) const { return h / t; }
  bool touches(int a, int b, int lo, int hi) const {
    for (int k = -40; k <= 40; ++k)
      if (a + k * n <= hi && b + k * n >= lo) return true;
    return false;
  }
  int needed(int h, int c) const {
    if (tile_of(h) == c) return 0;
    const int lo = first(c), hi = lo + width(c) - 1, m = mk ? 1 : 0;
    if (touches(h - 1 - m, h + 2 + m, fused ? lo - 1 - m : lo, fused ? hi + 2 + m : hi)) return 1;
    return touches(h - 1, h + 2, lo - 1 - R, hi + 1 + R) ? 2 : 3;
  }
};

static WorldDev world(const Axis& x, const Axis& y) {
  WorldDev w = {};
  static float some;
  w.nx = x.n;
  w.ny = y.n;
  w.ntx = x.nt;
  w.nty = y.nt;
  w.radius = x.R;
  w.tile_shift = tile_shift_of_side(x.t);
  w.tl_near = near_reach(x.mk, x.fused);
  if (x.mk) w.d_marker = &some;
  return w;
}
static Axis axis(int n, int t, int R, bool mk, bool fused) { return Axis{n, t, (n + t - 1) / t, R, mk, fused}; }

static int short_way(const Axis& x, int h, int c) {
  int best = 1 << 20;
  const int lo = x.first(c), w = x.width(c);
  for (int k = -1; k <= 1; ++k) {
    const int l = h + k * x.n - lo, out = l < 0 ? -l : (l >= w ? l - w + 1 : 0);
    if (out < (best < 0 ? -best : (best >= w ? best - w + 1 : 0))) best = l;
  }
  return best;
}
static bool in_span(const Axis& x, int at, int c) {   // the tiles that a tile reads the own nodes of
  const int s = axis_span(at, x.nt, x.t, x.n - (x.nt - 1) * x.t), m = min(2 * s + 1, x.nt);
  for (int i = 0; i < m; ++i)
    if ((m < x.nt ? wrap_near(at - s + i, x.nt) : i) == c) return true;
  return false;
}

template <int T>
static void one_axis(int n_max) {
  std::set<int> seen;                            // class triples of an axis, for the pairs below
  for (int n = 4; n <= n_max; ++n)
    for (int R = 1; R <= kMaxRadius; ++R)
      for (int opt = 0; opt < 4; ++opt) {
        const Axis x = axis(n, T, R, opt & 1, opt & 2), y = axis(T, T, R, opt & 1, opt & 2);
        const WorldDev w = world(x, y);
        const Reach reach(w);
        for (int h = 0; h < n; ++h) {
          std::vector<int> need(x.nt), got(x.nt, 3);
          for (int c = 0; c < x.nt; ++c) {
            std::snprintf(where, sizeof where, "n %d tile %d R %d markers %d fused %d home %d tile %d", n, T, R, opt & 1, opt >> 1, h, c);
            need[c] = x.needed(h, c);
            const int k = reach.of_cell(h, x.first(c), x.width(c), n);
            CHECK(k <= need[c] && (k == 0) == (need[c] == 0));
          }
          for_reached_tiles<T>(w, h, 0, [&](int tx, int, int k) { got[tx] = k; });
          for (int c = 0; c < x.nt; ++c) CHECK(got[c] <= need[c]);
          for (int c = 0; c < x.nt; ++c) {
            std::snprintf(where, sizeof where, "n %d tile %d R %d markers %d fused %d home %d left %d", n, T, R, opt & 1, opt >> 1, h, c);
            const Place p(w, T, c, 0, h, 0);
            const int width = x.width(c);
            const bool jump = p.lx < -kSmallMove || p.lx >= width + kSmallMove;
            const int l = short_way(x, h, c), far_out = l < 0 ? -l : (l >= width ? l - width + 1 : 0);
            CHECK(jump || far_out <= kSmallMove);   // (also where it is farther than that the way it is looked at)
            CHECK(!jump || !p.inside);
            if (!jump)
              for (int at = 0; at < x.nt; ++at) CHECK(need[at] > 2 || in_span(x, at, c));
            const Classes k = neighbour_classes<T>(w, c, 0, h, 0);
            CHECK(k.beyond == !p.inside);
            for (int at = 0; at < x.nt; ++at)
              if (p.inside && !next_to(w, c, 0, at, 0)) CHECK(need[at] == 3);
            for (int d = -1; d <= 1; ++d) {
              const int of = (k.kx >> (2 * d + 2)) & 3;
              if (!nb_exists(d, x.nt)) {
                CHECK(of == 3);
                continue;
              }
              const int want = need[nb_tile(c, d, x.nt)];
              CHECK(of <= want && (of == 0) == (want == 0));
            }
            seen.insert(k.kx);
          }
        }
      }
  for (int kx : seen)
    for (int ky : seen) {
      Classes c;
      c.kx = kx;
      c.ky = ky;
      c.beyond = false;
      std::snprintf(where, sizeof where, "tile %d classes %d %d", T, kx, ky);
      const Pairs a(c);
      if (a.more) continue;
      for (int q = 0; q < 8; ++q) {
        const int k = q == a.qx() ? a.side_x : q == a.qy() ? a.side_y : q == a.qc() ? a.corner : 3;
        CHECK(nb_dx(a.qx()) == a.dx && nb_dy(a.qy()) == a.dy && nb_dx(a.qc()) == a.dx && nb_dy(a.qc()) == a.dy);
        CHECK(k == c.of(q));
      }
    }
}

// Every node of a world, from each tile that it can have been listed by: all
// tiles that it reaches get it, each once.
template <int T>
static void two_axes(int nx, int ny, int R, bool mk, bool fused) {
  const Axis x = axis(nx, T, R, mk, fused), y = axis(ny, T, R, mk, fused);
  const WorldDev w = world(x, y);
  std::vector<int> got(x.nt * y.nt), times(x.nt * y.nt);
  for (int hy = 0; hy < ny; ++hy)
    for (int hx = 0; hx < nx; ++hx)
      for (int cy = 0; cy < y.nt; ++cy)
        for (int cx = 0; cx < x.nt; ++cx) {
          std::snprintf(where, sizeof where, "%d x %d tile %d R %d markers %d fused %d home %d %d left %d %d", nx, ny, T, R, mk, fused,
                        hx, hy, cx, cy);
          got.assign(got.size(), 3);
          times.assign(times.size(), 0);
          const auto put = [&](int tx, int ty, int k) {
            got[ty * x.nt + tx] = k;
            ++times[ty * x.nt + tx];
          };
          const Classes c = neighbour_classes<T>(w, cx, cy, hx, hy);
          put(cx, cy, 0);                        // its own nodes
          for (int q = 0; q < 8; ++q)
            if (c.of(q) <= 2) put(nb_tile(cx, nb_dx(q), x.nt), nb_tile(cy, nb_dy(q), y.nt), c.of(q));
          if (c.beyond)
            for_reached_tiles<T>(w, hx, hy, [&](int tx, int ty, int) {
              if (!next_to(w, cx, cy, tx, ty)) put(tx, ty, 0);
            });
          for (int ty = 0; ty < y.nt; ++ty)
            for (int tx = 0; tx < x.nt; ++tx) {
              const int need = max(x.needed(hx, tx), y.needed(hy, ty));
              CHECK(got[ty * x.nt + tx] <= need && times[ty * x.nt + tx] <= 1);
            }
        }
}

template <int T>
static void all(int n_max, int step) {
  one_axis<T>(n_max);
  const int sizes[][2] = {{T, T}, {T - 1, 2 * T}, {2 * T + 1, 3 * T}, {3 * T + 3, T + 2}, {4 * T + 9, 2 * T + 7}};
  for (const auto& s : sizes)
    for (int R = 1; R <= kMaxRadius; R += step)
      for (int opt = 0; opt < 4; ++opt) two_axes<T>(s[0], s[1], R, opt & 1, opt & 2);
}

int main(int argc, char** argv) {
  const int t = argc > 1 ? std::atoi(argv[1]) : 16;
  if (t == 16) all<16>(16 * 6 + 15, 7);
  else all<32>(32 * 5 + 31, 7);
  std::printf("%ld checks\n", n_checks);
  return 0;
}
