// Device helpers shared by the forward and adjoint kernels.
#pragma once

#include <math.h>

#include <type_traits>
#include <utility>

#include "engine.h"
#include "list_geometry.h"

namespace mc {

constexpr float kPi = 3.14159265358979323846f;
constexpr float kTwoPi = 6.28318530717958647692f;

// f(0), ..., f(N - 1) with compile-time arguments (integral constants): arrays
// indexed by them stay in registers.
template <int... I, class F>
static __device__ __forceinline__ void static_for_seq(std::integer_sequence<int, I...>, F f) {
  (f(std::integral_constant<int, I>()), ...);
}
template <int N, class F>
static __device__ __forceinline__ void static_for(F f) {
  static_for_seq(std::make_integer_sequence<int, N>(), f);
}

// i mod n in [0, n) for any i; integer division only outside [-n, 2n).
static __device__ __forceinline__ int wrap_index(int i, int n) {
  if (i >= 0 && i < n) return i;
  if (i >= n && i < 2 * n) return i - n;
  if (i < 0 && i >= -n) return i + n;
  const int r = i % n;
  return r < 0 ? r + n : r;
}

// Compile-time shape of the tile kernels for tiles of side TILE.
template <int TILE>
struct TileCfg {
  static constexpr int kTile = TILE;
  static constexpr int kShift = tile_shift_of_side(TILE);
  static constexpr int kFamily = tile_family_of_side(TILE);
  static constexpr int kThreads = TILE == 64 ? 1024 : 256;   // threads per tile block
  static constexpr bool kBinned = TILE < 64;                 // (64-cell tiles: sorted and direct worlds alone)
};

// Tile table entry it of a tile family: (world, tx | ty << 16); computed
// rather than read when the family holds a single world.
template <int TILE>
static __device__ __forceinline__ int2 tile_entry(const Tables& T, int it) {
  constexpr int f = TileCfg<TILE>::kFamily;
  if (T.single_ntx[f] > 0) {
    const int ty = it / T.single_ntx[f];
    return make_int2(0, (it - ty * T.single_ntx[f]) | (ty << 16));
  }
  return T.tiles[f][it];
}
template <int TILE>
static __device__ __forceinline__ int n_tiles(const Tables& T) {
  return *T.n_tiles[TileCfg<TILE>::kFamily];
}

// Tile table entries hold (world, tx | ty << 16).
static __device__ __forceinline__ int tile_x(int packed) { return packed & 0xffff; }
static __device__ __forceinline__ int tile_y(int packed) { return packed >> 16; }

// Map an angle difference into (-pi, pi] (the quotient by 2 pi is formed
// with its reciprocal; that can only matter at the boundary itself).
static __device__ __forceinline__ float wrap_angle(float d) {
  return d - kTwoPi * ceilf((d - kPi) * (1.0f / kTwoPi));
}

// Hardware square root and reciprocal (within 1 ulp; the edge lengths they
// see are near 1, far from denormals).
static __device__ __forceinline__ float hw_sqrt(float x) { return __builtin_amdgcn_sqrtf(x); }
static __device__ __forceinline__ float hw_rcp(float x) { return __builtin_amdgcn_rcpf(x); }

// The four 1D weights of Peskin's 4-point function for offsets
// (-1 - f, -f, 1 - f, 2 - f), f in [0, 1): with q = sqrt(1 + 4f - 4f^2) they
// are (3 - 2f - q)/8, (3 - 2f + q)/8, (1 + 2f + q)/8, (1 + 2f - q)/8.
// The square root's argument lies in [1, 2], where the hardware square root
// (within 1 ulp) needs none of the scaling of the library's sqrtf.
static __device__ __forceinline__ float peskin_q(float f) {
  return __builtin_amdgcn_sqrtf(fmaf(4.0f * f, 1.0f - f, 1.0f));
}
static __device__ __forceinline__ void peskin4(float f, float w[4]) {
  const float q = peskin_q(f);
  const float a = 3.0f - 2.0f * f;
  const float b = 1.0f + 2.0f * f;
  w[0] = 0.125f * (a - q);
  w[1] = 0.125f * (a + q);
  w[2] = 0.125f * (b + q);
  w[3] = 0.125f * (b - q);
}

// Derivatives of the four weights above with respect to f:
// with q' = (2 - 4f)/q they are (-2 - q')/8, (-2 + q')/8, (2 + q')/8, (2 - q')/8.
static __device__ __forceinline__ void peskin4_d(float f, float w[4], float dw[4]) {
  const float q = peskin_q(f);
  const float a = 3.0f - 2.0f * f;
  const float b = 1.0f + 2.0f * f;
  w[0] = 0.125f * (a - q);
  w[1] = 0.125f * (a + q);
  w[2] = 0.125f * (b + q);
  w[3] = 0.125f * (b - q);
  const float qd = (2.0f - 4.0f * f) / q;
  dw[0] = 0.125f * (-2.0f - qd);
  dw[1] = 0.125f * (-2.0f + qd);
  dw[2] = 0.125f * (2.0f + qd);
  dw[3] = 0.125f * (2.0f - qd);
}

// Actuated rest angle of joint j (of m: n - 2 on a chain, n on a loop) of a
// filament at time step t: ra + amp sin(2 pi t / period + phase - 2 pi j / m).
// The phase is formed in revolutions and reduced to [-1/2, 1/2] (the integer
// part of t / period is removed in FP64), so FP32 sinf sees a small argument.
static __device__ __forceinline__ float actuated_angle(float ra, float amp, float period, float phase, long long t,
                                                       int j, int m) {
  if (amp == 0.0f) return ra;
  float frac_t;                                 // (t / period) mod 1
  if (t < (1ll << 24)) {
    // t is exact in FP32; t - k period is formed with one rounding (fma), so
    // the remainder keeps FP32 accuracy whatever the size of t / period
    const float tf = (float)t;
    const float k = floorf(tf * hw_rcp(period));
    float rem = fmaf(-k, period, tf);
    if (rem < 0.0f) rem += period;
    if (rem >= period) rem -= period;
    frac_t = rem * hw_rcp(period);
  } else {
    const double q = (double)t / (double)period;
    frac_t = (float)(q - floor(q));
  }
  float r = frac_t + phase * (1.0f / kTwoPi) - (float)j / (float)m;
  r -= rintf(r);
  return ra + amp * sinf(kTwoPi * r);
}

// (cos t, sin t) of an edge angle t that started the step at t0, whose unit
// vector (c0, s0) is known: the rotation of (c0, s0) by d = t - t0, with
// cos d and sin d from their Taylor series (to d^8 and d^9; truncation below
// 3e-8 for |d| <= pi/4).  Larger turns take sincosf.
static __device__ __forceinline__ void edge_direction(float t, float t0, float c0, float s0, float* c, float* s) {
  const float d = t - t0;
  if (fabsf(d) <= 0.25f * kPi) {
    const float d2 = d * d;
    const float cd = fmaf(d2, fmaf(d2, fmaf(d2, fmaf(d2, 1.0f / 40320.0f, -1.0f / 720.0f), 1.0f / 24.0f), -0.5f), 1.0f);
    const float sd = d * fmaf(d2, fmaf(d2, fmaf(d2, fmaf(d2, 1.0f / 362880.0f, -1.0f / 5040.0f), 1.0f / 120.0f),
                                       -1.0f / 6.0f), 1.0f);
    *c = c0 * cd - s0 * sd;
    *s = s0 * cd + c0 * sd;
  } else {
    sincosf(t, s, c);
  }
}

// A marker displaced by d (|d| <= 1 cell) along one axis from a node with
// fraction f: the shift of its home cell from the node's (-1, 0 or 1) and
// its own fraction.  The shift stays in [-1, 1] also where |d| exceeds one
// cell by a rounding step: f + d rounded up to 2 is the same point as shift
// 1 with fraction 1 (the 4-point weights of fraction 1 put nothing on the
// first cell); f + d below -1 (by rounding only) moves to shift -1,
// fraction 0, at most one rounding step away.
static __device__ __forceinline__ void marker_shift(float f, float d, int* shift, float* fr) {
  const float m = f + d;
  const float fl = floorf(m);
  int h = (int)fl;
  float r = m - fl;
  if (r >= 1.0f) {
    r = 0.0f;
    h += 1;
  }
  if (h > 1) {
    h = 1;
    r = 1.0f;
  } else if (h < -1) {
    h = -1;
    r = 0.0f;
  }
  *shift = h;
  *fr = r;
}

// The same marker's wrapped home cell on an axis of n cells, for a node at cell c.
static __device__ __forceinline__ void marker_home(int c, float f, float d, int n, int* home, float* fr) {
  int sh;
  marker_shift(f, d, &sh, fr);
  *home = wrap_index(c + sh, n);
}

// Global float atomics of s * W(c - X) * (vx, vy) into an interleaved
// float2 field, for a point X with wrapped home cell (bx, by) and fraction (fx, fy).
static __device__ __forceinline__ void atomic_spread_vec(MC_GLOBAL float* field, int nx, int ny, int bx, int by,
                                                         float fx, float fy, float vx, float vy) {
  float wx[4], wy[4];
  peskin4(fx, wx);
  peskin4(fy, wy);
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    MC_GLOBAL float* row = field + 2 * (size_t)wrap_near(by - 1 + b, ny) * nx;
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      const int x = wrap_near(bx - 1 + a, nx);
      const float ww = wx[a] * wy[b];
      unsafeAtomicAdd((float*)(row + 2 * x), ww * vx);
      unsafeAtomicAdd((float*)(row + 2 * x + 1), ww * vy);
    }
  }
}

// sum_c W(c - X) v_c of an interleaved float2 field at a point X.
static __device__ __forceinline__ vf2 gather_vec(const MC_GLOBAL vf2* field, int nx, int ny, int bx, int by, float fx,
                                                 float fy) {
  float wx[4], wy[4];
  peskin4(fx, wx);
  peskin4(fy, wy);
  float gx = 0.f, gy = 0.f;
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    const MC_GLOBAL vf2* row = field + (size_t)wrap_near(by - 1 + b, ny) * nx;
    float ax = 0.f, ay = 0.f;
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      const vf2 v = row[wrap_near(bx - 1 + a, nx)];
      ax += wx[a] * v.x;
      ay += wx[a] * v.y;
    }
    gx += wy[b] * ax;
    gy += wy[b] * ay;
  }
  const vf2 out = {gx, gy};
  return out;
}

// D2Q9 lattice: velocity q has components (CX[q], CY[q]); q and q+2 are
// opposite for q = 1, 2, 5, 6.
static __constant__ int kCX[9] = {0, 1, 0, -1, 0, 1, -1, -1, 1};
static __constant__ int kCY[9] = {0, 0, 1, 0, -1, 1, 1, -1, -1};

// 64-bit fixed-point accumulation in LDS (2^-36 resolution, range +-2^27).
constexpr float kFixScale = 68719476736.0f;           // 2^36
constexpr float kFixInv = 1.4551915228366852e-11f;    // 2^-36
// Nearest 64-bit integer to a float x with |x| < 2^62, from 32-bit
// conversions: |x| = hi 2^32 + lo, where hi = floor(|x| / 2^32) and
// lo = |x| - hi 2^32 in [0, 2^32) are both exact in FP32 (|x| has 24
// significant bits, and so do its bits below 2^32), and lo only has a
// fraction when it is below 2^24.
static __device__ __forceinline__ long long f32_to_fix(float x) {
  const float ax = fabsf(x);
  const float hf = floorf(ax * 2.3283064365386963e-10f);
  const float lof = fmaf(hf, -4294967296.0f, ax);
  const long long m = (long long)(((unsigned long long)(unsigned)hf << 32) + (unsigned long long)__float2uint_rn(lof));
  return x < 0.0f ? -m : m;
}
static __device__ __forceinline__ float fix_to_float(long long v) {
  const int hi = (int)(v >> 32);
  const unsigned lo = (unsigned)v;
  return (float)((double)hi * 4294967296.0 + (double)lo) * kFixInv;
}

// Density deposits use the 1D weights rounded to multiples of 2^-23 (each
// weight is at most 1/2, so it is an integer below 2^23): a 2D weight is then
// the exact product of two such integers, a multiple of 2^-46 formed by two
// 24-bit multiplies, and sums of them are exact in 64 bits.
constexpr float kWeightQ = 8388608.0f;                   // 2^23
static __device__ __forceinline__ void peskin4_quant(float f, unsigned q[4]) {
  float w[4];
  peskin4(f, w);
#pragma unroll
  for (int a = 0; a < 4; ++a) q[a] = __float2uint_rn(w[a] * kWeightQ) & 0xffffffu;
}
static __device__ __forceinline__ unsigned long long weight_product(unsigned a, unsigned b) {
  return (unsigned long long)(a & 0xffffffu) * (b & 0xffffffu);   // v_mul_u32_u24 + v_mul_hi_u32_u24
}
// The high word converts exactly (densities stay far below 2^14), the low
// word with one FP32 rounding (an absolute error below 2^-38), then one fma.
static __device__ __forceinline__ float density_to_float(unsigned long long v) {
  return fmaf((float)(unsigned)(v >> 32), 6.103515625e-05f, (float)(unsigned)v * 1.4210854715202004e-14f);
}

// Work-item order of the tile kernels.  The hardware hands workgroups to the
// eight XCDs in turn (block b to XCD b mod 8) and each XCD has its own L2, so
// a plain grid-stride loop puts neighbouring tiles, which read each other's
// halos and list segments, on different XCDs.  Here the blocks of each XCD take one
// contiguous share of the item list instead.
struct XcdLoop {
  int first, end, step;
  __device__ __forceinline__ explicit XcdLoop(int n) : XcdLoop(n, blockIdx.x, gridDim.x) {}
  // block b of G (b mod 8 its XCD) of a list of n items
  __device__ __forceinline__ XcdLoop(int n, int b, int G) {
    if (G < 8) {
      first = b;
      end = n;
      step = G;
      return;
    }
    const int x = b & 7, per = (n + 7) >> 3;
    first = x * per + (b >> 3);
    end = min(n, x * per + per);
    step = (G - x + 7) >> 3;                   // blocks on this XCD
  }
};

// Clear n 64-bit words of LDS at a 16-byte aligned address, 16 bytes per
// store (block-wide; the caller synchronises before use).
static __device__ __forceinline__ void zero_lds_u64(void* p, int n) {
  vi4* q = (vi4*)p;
  const vi4 z = {0, 0, 0, 0};
  for (int k = threadIdx.x; k < (n >> 1); k += blockDim.x) q[k] = z;
  if ((n & 1) && threadIdx.x == 0) ((long long*)p)[n - 1] = 0;
}

// The lanes with `has` that share a lane's key: their first lane, their number
// and the lane's rank among them.  Formed by every active lane at once, so that
// all groups' atomics can be issued before the first result is waited for.
struct AggGroup {
  int leader, count, rank;
  __device__ __forceinline__ AggGroup(int key, bool has) : leader(__lane_id()), count(0), rank(0) {
    const int lane = __lane_id();
    unsigned long long pending = __ballot(has);
    while (pending) {
      const int first = __ffsll(pending) - 1;
      const int k = __shfl(key, first);
      const unsigned long long match = __ballot(has && key == k) & pending;
      if ((match >> lane) & 1ull) {
        leader = first;
        count = __popcll(match);
        rank = __popcll(match & ((1ull << lane) - 1ull));
      }
      pending &= ~match;
    }
  }
};

// Block-wide exclusive scan of one int per thread (NT threads), wave
// shuffles plus one LDS exchange (s_wave holds NT/64 ints).  Returns the
// exclusive prefix; *total gets the block sum.  All threads must call it.
template <int NT>
static __device__ __forceinline__ int block_scan(int v, int* s_wave, int* total) {
  const int lane = __lane_id();
  const int wid = threadIdx.x >> 6;
  int x = v;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int n = __shfl_up(x, off);
    if (lane >= off) x += n;
  }
  if (lane == 63) s_wave[wid] = x;
  __syncthreads();
  int before = 0, all = 0;
#pragma unroll
  for (int k = 0; k < NT / 64; ++k) {
    const int sw = s_wave[k];
    before += (k < wid) ? sw : 0;
    all += sw;
  }
  __syncthreads();
  *total = all;
  return before + x - v;
}
static __device__ __forceinline__ int block_scan256(int v, int* s_wave, int* total) {
  return block_scan<256>(v, s_wave, total);
}


// ---------------------------------------------------------------------------
// Tile lists (binned worlds; their layout: WorldDev).  A tile's list holds a
// record of every node its kernels need, once each.  Where a segment overflowed,
// the tile reads the own nodes of the tiles around it, which hold every node of
// theirs once; a world without lists is read by testing every node.
// ---------------------------------------------------------------------------
// Place of segment `seg` in a tile's list and its capacity (strays and own
// nodes come first, then the sides, then the corners, near before far).
static __device__ __forceinline__ int segment_first(const WorldDev& w, int seg) {
  if (seg < kCntNear) return seg == kCntOwn ? w.tl_strays : 0;
  const int q = (seg - kCntNear) & 7, s = w.tl_near_s + w.tl_far_s, c = w.tl_near_c + w.tl_far_c;
  return w.tl_strays + w.tl_own + (q < 4 ? q * s : 4 * s + (q - 4) * c) + (seg < kCntFar ? 0 : (q < 4 ? w.tl_near_s : w.tl_near_c));
}
static __device__ __forceinline__ int segment_cap(const WorldDev& w, int seg) {
  if (seg < kCntNear) return seg == kCntOwn ? w.tl_own : w.tl_strays;
  const int q = (seg - kCntNear) & 7;
  return seg < kCntFar ? (q < 4 ? w.tl_near_s : w.tl_near_c) : (q < 4 ? w.tl_far_s : w.tl_far_c);
}

// A tile's list counts (block-uniform: scalar loads; nothing in a kernel that
// reads them writes them).
typedef const __attribute__((address_space(4))) int* ListCounts;
static __device__ __forceinline__ ListCounts list_counts(const WorldDev& w, int tile) {
  return (ListCounts)(const int*)w.tl_cnt + (size_t)tile * kListCounts;
}

// Where a tile's nodes are read.  (What few tiles take is marked as unexpected,
// here and where lists are made: the kernels that use lists have more code than
// the instruction cache keeps from one launch to the next, and what most tiles
// run then lies together.  40,000 nodes on 640^2 30.9 -> 30.1 us per step, 12,000
// on 400^2 21.0 -> 20.8.)
enum ListMode : int {
  kModeList = 0,     // its list
  kModeAround = 1,   // the own nodes of the tiles around it
  kModeAll = 2       // every node of the world
};

// The runs of records that one wavefront of a block takes from a tile's list,
// all in scalar registers: its share of the strays and own nodes and (SEGS 2)
// the near and (3) the far nodes of one side and one corner neighbour, shared
// by the wavefronts that have the same pair.  Alone (SEGS 1), the own nodes go
// out in rounds of 64, so that one wavefront and not all has the last, short
// round.  Flat record f is record f + d[j], j the last run with pre[j] <= f.
// Other modes have one run at a time, d0 its first entry (kModeAround: the own
// nodes of every kWaves-th tile around; kModeAll: a part of the nodes).
template <int NT, int SEGS>
struct WaveRuns {
  static constexpr int kWaves = NT / 64;
  int mode, total;
  int p1, p2, p3, p4;                            // pre of runs 1 .. (SEGS 3: 4, else 2)
  int d0, e1, e2, e3, e4;                        // d of run 0, and what each run adds to the one before
  int next;                                      // kModeAround: this wavefront's next tile around
  bool outgrows;                                 // a segment that the tile's block writes may outgrow its place
  // record number of flat record f (clamped by the caller to [0, total))
  __device__ __forceinline__ int record(int f) const {
    int x = f + d0;
    if constexpr (SEGS > 1) x += (f >= p1 ? e1 : 0) + (f >= p2 ? e2 : 0);
    if constexpr (SEGS == 3) x += (f >= p3 ? e3 : 0) + (f >= p4 ? e4 : 0);
    return x;
  }
  // The next tile around that has own nodes (kModeAround); false: no more.
  __device__ __forceinline__ bool next_run(const WorldDev& w, int tile) {
    const int ntx = w.ntx, nty = w.nty, side = 1 << w.tile_shift, ty = tile / ntx, tx = tile - ty * ntx;
    const int sx = axis_span(tx, ntx, side, w.nx - (ntx - 1) * side), sy = axis_span(ty, nty, side, w.ny - (nty - 1) * side);
    const int mx = min(2 * sx + 1, ntx), my = min(2 * sy + 1, nty);
    total = 0;
    while (next < mx * my) {
      const int j = next / mx, i = next - j * mx;
      next += kWaves;
      const ListCounts c = list_counts(w, (my < nty ? wrap_near(ty - sy + j, nty) : j) * ntx +
                                              (mx < ntx ? wrap_near(tx - sx + i, ntx) : i));
      total = c[kCntOwn];
      d0 = c[kFirst + kCntOwn];
      if (total > 0) return true;
    }
    return false;
  }
};
// The part of the wavefronts that share n records: number `part` of `of`.
struct RunPart {
  int a, n;
  __device__ __forceinline__ RunPart(int all, int part, int of) : a(all * part / of), n(all * (part + 1) / of - a) {}
  __device__ __forceinline__ RunPart(int a, int n) : a(a), n(n) {}
};
// The same in rounds of 64.
static __device__ __forceinline__ RunPart round_part(int all, int part, int of) {
  const int rounds = (int)((unsigned)(all + 63) >> 6), each = rounds / of, more = rounds % of;
  const int a = min(64 * (part * each + min(part, more)), all);
  return RunPart(a, min(64 * (each + (part < more ? 1 : 0)), all - a));
}
// A neighbour's segments as runs: near nodes, far nodes.
template <int SEGS>
static __device__ __forceinline__ void neighbour_runs(int ntx, int nty, ListCounts c, int q, int* first, int* n,
                                                      int* far_first, int* far_n) {
  *first = *n = *far_first = *far_n = 0;
  if (!nb_exists(nb_dx(q), ntx) || !nb_exists(nb_dy(q), nty)) return;       // (nobody writes its numbers)
  *first = c[kFirst + kCntNear + q];
  *n = c[kCntNear + q];
  if (SEGS == 3) {
    *far_first = c[kFirst + kCntFar + q];
    *far_n = c[kCntFar + q];
  }
}
template <int NT, int SEGS>
static __device__ __forceinline__ WaveRuns<NT, SEGS> wave_runs(const WorldDev& w, int tile) {
  constexpr int kWaves = NT / 64, kShare = kWaves / 4;
  static_assert(kWaves % 4 == 0, "four neighbour pairs");
  int mode = kModeAll, strays = 0, own = 0, first = 0, fs = 0, ns = 0, ffs = 0, nfs = 0, fc = 0, nc = 0, ffc = 0, nfc = 0;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), pair = kWaves == 4 ? wave : wave & 3,
            share = kWaves == 4 ? 0 : wave >> 2;
  // (what the list's place needs of the world, in one round of loads: 12,800 nodes
  // on 256^2 19.5 -> 19.2 us per step)
  int kind = w.tl_kind, own_cap = w.tl_own, stray_cap = w.tl_strays, stride = w.tl_stride, ntx = w.ntx, nty = w.nty;
  const int* cnt = w.tl_cnt;
  asm volatile("" : "+s"(kind), "+s"(own_cap), "+s"(stray_cap), "+s"(stride), "+s"(ntx), "+s"(nty), "+s"(cnt));
  const ListCounts c = (ListCounts)cnt + (size_t)tile * kListCounts;
  bool outgrows = false;
  if (kind != kNoLists) {
    int flags = c[kCntFlags], crowded = c[kCntCrowded];
    strays = c[kCntStrays];
    own = c[kCntOwn];
    first = c[kFirst + kCntOwn];
    if constexpr (SEGS > 1) {
      neighbour_runs<SEGS>(ntx, nty, c, pair, &fs, &ns, &ffs, &nfs);
      neighbour_runs<SEGS>(ntx, nty, c, pair + 4, &fc, &nc, &ffc, &nfc);
    }
    // (everything is asked for before the flags are waited for)
    asm volatile("" : "+s"(flags), "+s"(crowded), "+s"(strays), "+s"(own), "+s"(first), "+s"(ns), "+s"(nc));
    outgrows = crowded || own + strays > own_cap;
    if (kind == kSegments && !(flags & (SEGS > 1 ? ~0 : kOverStrays | kOverOwn))) mode = kModeList;
    else if (!(flags & kOverOwn) && !((ListCounts)cnt + (size_t)(ntx * nty) * kListCounts)[kWordJump]) mode = kModeAround;
  }
  if (mode == kModeAll) {
    const RunPart r = round_part(w.n_part, wave, kWaves);
    return {mode, r.n, 0, 0, 0, 0, r.a, 0, 0, 0, 0, 0, outgrows};
  }
  if (__builtin_expect(mode == kModeAround, 0)) {
    WaveRuns<NT, SEGS> L = {mode, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, wave, outgrows};
    L.next_run(w, tile);
    return L;
  }
  // strays and own nodes are one run, or where the own nodes lie in the spill
  // area two, the first of them for wavefront 0
  const int home = tile * stride + stray_cap, all = strays + own;
  const bool apart = first != home;
  RunPart r0 = SEGS == 1 ? round_part(all, wave, kWaves) : RunPart(all, wave, kWaves);
  int d0 = home - strays;
  if (__builtin_expect(apart, 0)) {
    r0 = wave == 0 ? RunPart(0, strays) : round_part(own, wave - 1, kWaves - 1);
    d0 = wave == 0 ? d0 : first;
  }
  if constexpr (SEGS == 1) {
    return {mode, r0.n, 0, 0, 0, 0, d0 + r0.a, 0, 0, 0, 0, 0, outgrows};
  } else {
    // (with some 20 more scalar instructions the own nodes go out so that the
    // wavefronts' totals fill as few rounds of 64 as the tile needs, in the
    // tiles where equal shares may take more: 8 rounds for 256 own nodes, now 6)
    if (kWaves == 4 && all > 128 && ntx > 2 && nty > 2 && !apart) {
      const auto pair_n = [&](int q) {
        return c[kCntNear + q] + c[kCntNear + q + 4] + (SEGS == 3 ? c[kCntFar + q] + c[kCntFar + q + 4] : 0);
      };
      const int n0 = pair_n(0), n1 = pair_n(1), n2 = pair_n(2), n3 = pair_n(3);
      const int rounds = (unsigned)(all + n0 + n1 + n2 + n3 + 63) >> 6, each = rounds >> 2, more = rounds & 3;
      const int a0 = max(64 * (each + (more > 0 ? 1 : 0)) - n0, 0), a1 = max(64 * (each + (more > 1 ? 1 : 0)) - n1, 0),
                a2 = max(64 * (each + (more > 2 ? 1 : 0)) - n2, 0);
      const int b1 = min(a0, all), b2 = min(a0 + a1, all), b3 = min(a0 + a1 + a2, all);
      r0.a = wave == 0 ? 0 : (wave == 1 ? b1 : (wave == 2 ? b2 : b3));
      r0.n = (wave == 0 ? b1 : (wave == 1 ? b2 : (wave == 2 ? b3 : all))) - r0.a;
    }
    const RunPart r1(ns, share, kShare), r2(nfs, share, kShare), r3(nc, share, kShare),
        r4(nfc, share, kShare);
    d0 += r0.a;
    const int p1 = r0.n, d1 = fs + r1.a - p1;
    if constexpr (SEGS == 3) {
      const int p2 = p1 + r1.n, d2 = ffs + r2.a - p2, p3 = p2 + r2.n, d3 = fc + r3.a - p3, p4 = p3 + r3.n,
                d4 = ffc + r4.a - p4;
      return {mode, p4 + r4.n, p1, p2, p3, p4, d0, d1 - d0, d2 - d1, d3 - d2, d4 - d3, 0, outgrows};
    } else {
      const int p2 = p1 + r1.n, d2 = fc + r3.a - p2;
      return {mode, p2 + r3.n, p1, p2, 0, 0, d0, d1 - d0, d2 - d1, 0, 0, 0, outgrows};
    }
  }
}

// The record of node i.
static __device__ __forceinline__ vi4 node_record(const WorldDev& w, int i) {
  const int N = w.n_part;
  const MC_GLOBAL int* cell = glb(w.cell_in);
  const MC_GLOBAL float* frac = glb(w.frac_in);
  const int hx = wrap_index(cell[i], w.nx), hy = wrap_index(cell[N + i], w.ny);
  const vi4 r = {hx | (hy << 16), __float_as_int(frac[i]), __float_as_int(frac[N + i]), i};
  return r;
}

// The records of a tile's list (SEGS as in WaveRuns) for the NT threads of a
// block, in any order, PER per thread in flight with the values v[node] (VALS
// 1) and v[N + node] (2) of their nodes.  The first round of a list is loaded
// where the object is made, so that its chain of loads (counts, records, values)
// runs beside what the block does before it needs them: at the sizes where a
// launch lasts as long as that chain, and where the blocks of a CU go through
// their phases together.
template <int NT, int SEGS, int PER, int VALS = 0>
struct TileRecords {
  const MC_GLOBAL float* v;
  WaveRuns<NT, SEGS> L;
  int N, tile;
  vi4 r[PER];
  vf2 val[PER];
  __device__ __forceinline__ vf2 value(int node) const {
    const vf2 x = {VALS > 0 ? v[node] : 0.f, VALS > 1 ? v[N + node] : 0.f};
    return x;
  }
  // The round from `base` of a list (clamped, so that every load is issued at once).
  __device__ __forceinline__ void load(const WorldDev& w, int base) {
    const MC_GLOBAL vi4* rec = glbv<const vi4>(w.tl_rec);
#pragma unroll
    for (int i = 0; i < PER; ++i) r[i] = rec[L.record(min(base + i * 64 + (int)(threadIdx.x & 63), L.total - 1))];
#pragma unroll
    for (int i = 0; i < PER; ++i) val[i] = value(r[i].w);
  }
  // Record of flat number f of another run.
  __device__ __forceinline__ vi4 run_record(const WorldDev& w, int f) const {
    const int e = L.d0 + f;
    if (__builtin_expect(L.mode == kModeAround && w.tl_kind != kOwnIndices, 0)) return glbv<const vi4>(w.tl_rec)[e];
    return node_record(w, L.mode == kModeAll ? e : glb((const int*)w.tl_rec)[e]);
  }
  __device__ __forceinline__ TileRecords(const WorldDev& w, int tile, const MC_GLOBAL float* values = nullptr)
      : v(values), L(wave_runs<NT, SEGS>(w, tile)), N(w.n_part), tile(tile) {
    if (L.mode == kModeList && L.total > 0) load(w, 0);
  }
  // body(record, value) for each.  body must itself drop the records its window
  // does not hold (the list may hold more than needed, and where it cannot be
  // used body gets other nodes too).  No barrier; body may only use per-lane
  // work and LDS atomics.
  template <class Body>
  __device__ __forceinline__ void each(const WorldDev& w, Body body) {
    if (__builtin_expect(L.mode == kModeList, 1)) {
      for (int base = 0; base < L.total; base += PER * 64) {
        if (base > 0) load(w, base);
#pragma unroll
        for (int i = 0; i < PER; ++i)
          if (base + i * 64 + (int)(threadIdx.x & 63) < L.total) body(r[i], val[i]);
      }
      return;
    }
    do {
      for (int f = threadIdx.x & 63; f < L.total; f += 64) {
        const vi4 q = run_record(w, f);
        body(q, value(q.w));
      }
    } while (L.mode == kModeAround && L.next_run(w, tile));
  }
};
// (what a tile spread goes through)
template <int TILE, bool SCALAR = false>
using SpreadNodes = TileRecords<TileCfg<TILE>::kThreads, 2, 2, SCALAR ? 1 : 2>;

// body(record) for the own nodes of the tile [x0, x0 + tw) x [y0, y0 + th).
template <int NT, class Body>
static __device__ __forceinline__ void for_own_records(const WorldDev& w, int tile, int x0, int y0,
                                                       int tw, int th, Body body) {
  TileRecords<NT, 1, 1> nodes(w, tile);
  nodes.each(w, [&](const vi4& r, const vf2&) {
    const int lx = (r.x & 0xffff) - x0, ly = (r.x >> 16) - y0;
    if (lx >= 0 && lx < tw && ly >= 0 && ly < th) body(r);
  });
}

// Node -> grid accumulation over a padded window.  A window of side
// S = need + 6 covers grid cells o + c (c in [0, S), o = origin, periodic)
// for a caller that reads the `need` cells [3, 3 + need); a node whose home
// cell is h adds to window cells d + (0..3), d = (h - 1 - o) mod n in [0, n).
// Every contribution lands inside the window, so the inner loops carry no
// bounds or wrap tests:
//   * when need + 3 <= n, a node with d > need + 2 cannot touch the needed
//     cells (its support lies past them, and the part that wraps lands in
//     cells 0..2), so only nodes with d <= need + 2 are kept: their cells
//     reach at most need + 5;
//   * otherwise (small grids, n < need + 3) every node of the list is kept,
//     its cells reach at most n + 2 < S, and window cells that are the same
//     grid cell are summed when read.
// The first three and last three window cells only catch the spill of nodes
// at the edge of the needed range.

// Window cell sum for needed cell i (window cell 3 + i) on an axis of n cells:
// one term unless the window wraps onto itself.
static __device__ __forceinline__ int first_image(int i, int n) {
  const int c = i + 3;
  return c < n ? c : c % n;
}

// A vector field over the SIDE x SIDE cells from (ox, oy) (periodic) on its way
// to LDS: every load is in flight once the object is made, store() waits for
// them.  No barrier.
template <int NT, int SIDE>
struct WindowLoads {
  static constexpr int kCells = SIDE * SIDE, kIt = (kCells + NT - 1) / NT;
  vf2 v[kIt];
  __device__ __forceinline__ WindowLoads(const MC_GLOBAL vf2* f, int nx, int ny, int ox, int oy) {
    const int wx = wrap_index(ox, nx), wy = wrap_index(oy, ny);
#pragma unroll
    for (int i = 0; i < kIt; ++i) {
      const int k = min((int)threadIdx.x + NT * i, kCells - 1);
      const int r = k / SIDE, c = k - (k / SIDE) * SIDE;
      v[i] = f[(size_t)wrap_index(wy + r, ny) * nx + wrap_index(wx + c, nx)];
    }
  }
  __device__ __forceinline__ void store(vf2* st) const {
#pragma unroll
    for (int i = 0; i < kIt; ++i) {
      const int k = (int)threadIdx.x + NT * i;
      if (k < kCells) st[k] = v[i];
    }
  }
};
// Tile spread: for every node whose 4x4 support meets the needed cells
// [x0 - LO, x0 + tw + HI) x [y0 - LO, y0 + th + HI) of the tile [x0, x0 + tw) x
// [y0, y0 + th), add scale * W(c - x_i) * (v[i], v[N + i]) to the window
// accumulators s_x, s_y (64-bit fixed point, side TILE + LO + HI + 6, origin
// (x0 - LO - 3, y0 - LO - 3)).  Nodes are read from the tile's own and near
// lists.  All threads of the block call it; the accumulators must be zeroed
// (and synchronised) beforehand, and the caller synchronises after it.
// Values whose fixed-point image fits 32 bits (|scale v| < 1/8, as nearly all
// forces) are converted by one truncating 32-bit conversion; larger ones by
// the exact 64-bit split.
template <int TILE, int LO = 0, int HI = 0>
struct SpreadWin {
  static constexpr int kSide = TILE + LO + HI + 6, kCells = kSide * kSide;
  static constexpr int kGSide = kSide + 2, kGCells = kGSide * kGSide;   // gradient of a two-layer world
};

// One point's 4x4 contribution W * (Vx, Vy) to two 64-bit fixed-point LDS
// windows of row length SIDE at the point's support origin (px, py).
template <int SIDE, bool SCALAR = false>
static __device__ __forceinline__ void spread_point(long long* sx, long long* sy, const float* wx,
                                                    const float* wy, float Vx, float Vy) {
  unsigned long long* px = (unsigned long long*)sx;
  unsigned long long* py = (unsigned long long*)sy;
  if (fmaxf(fabsf(Vx), fabsf(Vy)) < 0.125f) {
    float ax[4], ay[4];
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      ax[a] = (Vx * kFixScale) * wx[a];
      ay[a] = (Vy * kFixScale) * wx[a];
    }
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
      for (int a = 0; a < 4; ++a) {
        atomicAdd(px + b * SIDE + a, (unsigned long long)(long long)(int)(ax[a] * wy[b]));
        if constexpr (!SCALAR) atomicAdd(py + b * SIDE + a, (unsigned long long)(long long)(int)(ay[a] * wy[b]));
      }
  } else {
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
      for (int a = 0; a < 4; ++a) {
        const float ww = wx[a] * wy[b];
        atomicAdd(px + b * SIDE + a, (unsigned long long)f32_to_fix(ww * Vx * kFixScale));
        if constexpr (!SCALAR) atomicAdd(py + b * SIDE + a, (unsigned long long)f32_to_fix(ww * Vy * kFixScale));
      }
  }
}

// With s_g (REP), the spread value of a node is its total force: v (the
// elastic force) minus k_rep times the kernel-weighted gradient at its
// support, read from s_g, the gradient staged over the same window; the home
// tile of a node (the one tile holding its home cell) also writes that total
// to w.fel.  The gradient sum runs in the same order as the repulsion gather
// of the node kernels, so the forces are the same.  SCALAR spreads
// scale * v[i] alone into s_x (s_y is not touched and may be null).
template <int TILE, bool REP, bool SCALAR = false, int LO = 0, int HI = 0>
static __device__ __forceinline__ void tile_spread_vec(const WorldDev& w, SpreadNodes<TILE, SCALAR>& nodes, int x0,
                                                       int y0, int tw, int th, float scale,
                                                       long long* s_x, long long* s_y, const vf2* s_g) {
  constexpr int kSide = SpreadWin<TILE, LO, HI>::kSide;
  const int nx = w.nx, ny = w.ny, N = w.n_part;
  const int ox = wrap_index(x0 - LO - 3, nx), oy = wrap_index(y0 - LO - 3, ny);
  const int nw = tw + LO + HI, nh = th + LO + HI;
  const int keep_x = nw + 3 <= nx ? nw + 2 : nx;     // largest kept home offset
  const int keep_y = nh + 3 <= ny ? nh + 2 : ny;
  const float kr = w.k_rep;
  MC_GLOBAL float* ftot = glb(w.fel);
  nodes.each(w, [&](const vi4& r, const vf2& v) {
    const int dx = wrap_near((r.x & 0xffff) - 1 - ox, nx);
    const int dy = wrap_near((r.x >> 16) - 1 - oy, ny);
    if (dx > keep_x || dy > keep_y) return;
    float wx[4], wy[4];
    peskin4(__int_as_float(r.y), wx);
    peskin4(__int_as_float(r.z), wy);
    float Vx, Vy;
    if constexpr (REP) {
      float gx = 0.f, gy = 0.f;
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        const vf2* row = s_g + (dy + b) * kSide + dx;
        float ax = 0.f, ay = 0.f;
#pragma unroll
        for (int a = 0; a < 4; ++a) {
          const vf2 t = row[a];
          ax += wx[a] * t.x;
          ay += wx[a] * t.y;
        }
        gx += wy[b] * ax;
        gy += wy[b] * ay;
      }
      Vx = v.x - kr * gx;
      Vy = v.y - kr * gy;
      const int hx = r.x & 0xffff, hy = r.x >> 16;
      if (hx >= x0 && hx < x0 + tw && hy >= y0 && hy < y0 + th) {
        ftot[r.w] = Vx;
        ftot[N + r.w] = Vy;
      }
    } else {
      Vx = scale * v.x;
      Vy = SCALAR ? 0.f : scale * v.y;
    }
    spread_point<kSide, SCALAR>(s_x + dy * kSide + dx, s_y + dy * kSide + dx, wx, wy, Vx, Vy);
  });
}

// The tile spread of a two-layer world: each node acts through its markers
// X = x +- d (d from w.d_marker), each taking half of the node's value.  The
// node's value is formed as in tile_spread_vec, with the gradient s_g staged
// over a window one cell wider on every side (side kSide + 2, origin
// (x0 - LO - 4, y0 - LO - 4)), since a node whose marker reaches the needed
// cells can lie one cell further out.  The accumulators keep their side and
// origin: a marker goes in by the one-layer keep rule applied to its own home
// cell, and the others cannot touch the needed cells.
template <int TILE, bool REP, int LO = 0, int HI = 0>
static __device__ __forceinline__ void tile_spread_markers(const WorldDev& w, SpreadNodes<TILE>& nodes, int x0, int y0,
                                                           int tw, int th, float scale, long long* s_x, long long* s_y,
                                                           const vf2* s_g) {
  constexpr int kSide = SpreadWin<TILE, LO, HI>::kSide, kGSide = SpreadWin<TILE, LO, HI>::kGSide;
  const int nx = w.nx, ny = w.ny, N = w.n_part;
  const int ox = wrap_index(x0 - LO - 3, nx), oy = wrap_index(y0 - LO - 3, ny);
  const int gox = wrap_index(x0 - LO - 4, nx), goy = wrap_index(y0 - LO - 4, ny);
  const int nw = tw + LO + HI, nh = th + LO + HI;
  const int keep_x = nw + 3 <= nx ? nw + 2 : nx;     // markers: largest kept home offset
  const int keep_y = nh + 3 <= ny ? nh + 2 : ny;
  const int nkeep_x = nw + 5 <= nx ? nw + 4 : nx;    // nodes: one cell more on each side
  const int nkeep_y = nh + 5 <= ny ? nh + 4 : ny;
  const float kr = w.k_rep;
  MC_GLOBAL float* ftot = glb(w.fel);
  const MC_GLOBAL float* dm = glb(w.d_marker);
  nodes.each(w, [&](const vi4& r, const vf2& v) {
    const int hx = r.x & 0xffff, hy = r.x >> 16;
    const int dx = wrap_near(hx - 1 - gox, nx), dy = wrap_near(hy - 1 - goy, ny);
    if (dx > nkeep_x || dy > nkeep_y) return;
    const float fx = __int_as_float(r.y), fy = __int_as_float(r.z);
    float Vx, Vy;
    if constexpr (REP) {
      float wx[4], wy[4];
      peskin4(fx, wx);
      peskin4(fy, wy);
      float gx = 0.f, gy = 0.f;
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        const vf2* row = s_g + (dy + b) * kGSide + dx;
        float ax = 0.f, ay = 0.f;
#pragma unroll
        for (int a = 0; a < 4; ++a) {
          const vf2 t = row[a];
          ax += wx[a] * t.x;
          ay += wx[a] * t.y;
        }
        gx += wy[b] * ax;
        gy += wy[b] * ay;
      }
      Vx = v.x - kr * gx;
      Vy = v.y - kr * gy;
      if (hx >= x0 && hx < x0 + tw && hy >= y0 && hy < y0 + th) {
        ftot[r.w] = Vx;
        ftot[N + r.w] = Vy;
      }
    } else {
      Vx = scale * v.x;
      Vy = scale * v.y;
    }
    const float ddx = dm[r.w], ddy = dm[N + r.w];
    const float hVx = 0.5f * Vx, hVy = 0.5f * Vy;
#pragma unroll
    for (int l = 0; l < 2; ++l) {
      const float sg = l == 0 ? 1.f : -1.f;
      int sx, sy;
      float mx, my;
      marker_shift(fx, sg * ddx, &sx, &mx);
      marker_shift(fy, sg * ddy, &sy, &my);
      const int mdx = wrap_index(hx + sx - 1 - ox, nx), mdy = wrap_index(hy + sy - 1 - oy, ny);
      if (mdx <= keep_x && mdy <= keep_y) {
        float wx[4], wy[4];
        peskin4(mx, wx);
        peskin4(my, wy);
        spread_point<kSide>(s_x + mdy * kSide + mdx, s_y + mdy * kSide + mdx, wx, wy, hVx, hVy);
      }
    }
  });
}

// The accumulated value of needed cell (i, j) of a spread window of side SIDE.
template <int SIDE>
static __device__ __forceinline__ long long spread_cell(const long long* s, int i, int j, int nx, int ny) {
  const int cx0 = first_image(i, nx), cy0 = first_image(j, ny);
  if (cx0 + nx >= SIDE && cy0 + ny >= SIDE) return s[cy0 * SIDE + cx0];
  long long acc = 0;
  for (int cy = cy0; cy < SIDE; cy += ny)
    for (int cx = cx0; cx < SIDE; cx += nx) acc += s[cy * SIDE + cx];
  return acc;
}

template <int TILE>
static inline bool tile_family_present(const Grid& G) {
  return G.tile_blocks[TileCfg<TILE>::kFamily] > 0;
}

// Host side: launch a tile kernel with a one-layer and a two-layer variant
// (template argument MK last) for the tile families of binned worlds, in the
// variants the grid needs: launch(Int<TILE>, Bool<MK>) launches one.  Each
// variant skips the other's worlds; the two-layer one runs only where a
// binned world has markers, the one-layer one unless every world has them.
template <class L>
static inline void for_tile_variants(const Grid& G, L launch) {
  const bool mk = G.any_markers && G.any_binned, plain = !G.mk_only;
  if (tile_family_present<16>(G)) {
    if (plain) launch(std::integral_constant<int, 16>(), std::false_type());
    if (mk) launch(std::integral_constant<int, 16>(), std::true_type());
  }
  if (tile_family_present<32>(G)) {
    if (plain) launch(std::integral_constant<int, 32>(), std::false_type());
    if (mk) launch(std::integral_constant<int, 32>(), std::true_type());
  }
}

}  // namespace mc
