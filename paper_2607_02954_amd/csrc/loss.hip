// Objectives and descriptors computed from a world's state.
//
// Folding objective (Experiments, Filament Folding): the node density
// splatted with a Gaussian onto an image that covers the periodic world, its
// mean squared error to a target image, and the gradient of that loss with
// respect to the node positions.  Behavioural descriptors (Experiments, QD
// Search, Eqs. 5-6): bending and stretching effort of a change of the rest
// values, per filament.
//
// Pixel (a, b) of a W x H image is centred at world point
// (-1/2 + (a + 1/2) hx, -1/2 + (b + 1/2) hy), hx = nx / W, hy = ny / H; node i
// adds amp exp(-r^2 / (2 sigma^2)) to every pixel whose centre lies within
// r <= 5 sigma of it (periodic minimum-image distance).
//
//   k_splat_tile      per 8x8 tile of pixels: the nodes that reach it, their
//                     contributions summed per pixel as 64-bit fixed point
//                     (order-independent: bitwise reproducible); the image,
//                     2 (I - T) / P for the gradient, and the tile's sum of
//                     (I - T)^2 in a fixed order
//   k_splat_image     many nodes: per node, its pixels' contributions added to
//                     a global 64-bit fixed-point image, which
//   k_image_residual  turns into the same outputs per 256 pixels
//   k_splat_grad      dL/dx_i = sum over node i's pixels of
//                     2 (I - T) / P * amp e^{-r^2/2s^2} * (-(x_i - c) / s^2);
//                     its last block forms the loss from the block sums
//                     (fixed order)
#include <algorithm>
#include <cmath>

#include "device_util.h"

namespace mc {

constexpr float kImgFix = 1099511627776.0f;          // 2^40: image fixed-point scale
constexpr double kImgFixInv = 1.0 / 1099511627776.0;
constexpr int kLossBlock = 256;
struct SplatGeom {
  int nx, ny, n, W, H;
  float hx, hy;          // pixel spacing (cells)
  float inv2s2;          // 1 / (2 sigma^2)
  float inv_s2;          // 1 / sigma^2
  float cut2;            // (5 sigma)^2
  float reach;           // 5 sigma and its rounding, for whole tiles
  float amp;
  int rx, ry;            // pixel window half-widths; rx < 0: every column once (same for ry)
};

// Minimum-image difference d (|d| < 2n on entry) reduced to [-n/2, n/2).
static __device__ __forceinline__ float wrap_half(float d, float n) {
  if (d >= 0.5f * n) d -= n;
  if (d < -0.5f * n) d += n;
  return d;
}

// The pixels of node (xw, yw) (wrapped world position): calls f(pixel index,
// dx, dy, weight) for every pixel centre within the cutoff, each pixel once.
// LANES > 1: lane `sub` of LANES takes every LANES-th pixel of the window.
template <int LANES, class F>
static __device__ __forceinline__ void for_node_pixels(const SplatGeom& g, float xw, float yw, int sub, F f) {
  const int a0 = (int)floorf((xw + 0.5f) / g.hx);      // pixel column holding the node
  const int b0 = (int)floorf((yw + 0.5f) / g.hy);
  const int alo = g.rx < 0 ? 0 : a0 - g.rx, na = g.rx < 0 ? g.W : 2 * g.rx + 1;
  const int blo = g.ry < 0 ? 0 : b0 - g.ry, nb = g.ry < 0 ? g.H : 2 * g.ry + 1;
  int b = sub / na, a = sub - b * na;
  while (b < nb) {
    const int bw = wrap_index(blo + b, g.H), aw = wrap_index(alo + a, g.W);
    const float dy = wrap_half(yw - (-0.5f + ((float)bw + 0.5f) * g.hy), (float)g.ny);
    const float dx = wrap_half(xw - (-0.5f + ((float)aw + 0.5f) * g.hx), (float)g.nx);
    const float r2 = dx * dx + dy * dy;
    if (r2 <= g.cut2) f(bw * g.W + aw, dx, dy, g.amp * expf(-r2 * g.inv2s2));
    a += LANES;
    while (a >= na) {
      a -= na;
      ++b;
    }
  }
}

static __device__ __forceinline__ void node_position(const SplatGeom& g, const int* cell, const float* frac, int i,
                                                     float* xw, float* yw) {
  *xw = (float)wrap_index(cell[i], g.nx) + frac[i];
  *yw = (float)wrap_index(cell[g.n + i], g.ny) + frac[g.n + i];
}

__global__ void k_zero_u64(unsigned long long* p, int n) {
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) p[i] = 0ull;
}

template <int LANES>
__global__ __launch_bounds__(kLossBlock) void k_splat_image(SplatGeom g, const int* cell, const float* frac,
                                                            unsigned long long* acc) {
  const int per = kLossBlock / LANES, sub = threadIdx.x % LANES;
  for (int i = blockIdx.x * per + threadIdx.x / LANES; i < g.n; i += gridDim.x * per) {
    float xw, yw;
    node_position(g, cell, frac, i, &xw, &yw);
    for_node_pixels<LANES>(g, xw, yw, sub, [&](int pix, float, float, float v) {
      atomicAdd(acc + pix, (unsigned long long)f32_to_fix(v * kImgFix));
    });
  }
}

__global__ __launch_bounds__(kLossBlock) void k_image_residual(SplatGeom g, const unsigned long long* acc,
                                                               const float* target, float* image, float* resid,
                                                               float* partial) {
  __shared__ float s_sum[kLossBlock];
  const int P = g.W * g.H;
  const int p = blockIdx.x * kLossBlock + threadIdx.x;
  float e2 = 0.f;
  if (p < P) {
    const float I = (float)((double)(long long)acc[p] * kImgFixInv);
    const float r = I - target[p];
    if (image) image[p] = I;
    resid[p] = 2.0f * r / (float)P;
    e2 = r * r;
  }
  s_sum[threadIdx.x] = e2;
  __syncthreads();
  for (int off = kLossBlock / 2; off > 0; off >>= 1) {   // fixed pairing: deterministic
    if ((int)threadIdx.x < off) s_sum[threadIdx.x] += s_sum[threadIdx.x + off];
    __syncthreads();
  }
  if (threadIdx.x == 0) partial[blockIdx.x] = s_sum[0];
}

// The image tile by tile: every block tests all nodes against its tile
// (kSplatChunk at a time, the reaching ones compacted into LDS) and each
// wavefront sums a quarter of them, a lane per pixel, in registers: no atomics, no
// accumulator image to clear, and the residual in the same pass.  A thread
// per node adding its pixels to HBM by 64-bit atomics ran 1000 nodes on 128^2
// pixels as 4 blocks of long serial loops: 33 us, 4.7 for the residual and 3.9
// for the clearing; the 256 blocks here take about 7.  Bound by the chain of
// loads, compaction and barriers per kSplatChunk nodes.
constexpr int kImgTile = 8;
constexpr int kSplatChunk = 1024;
__global__ __launch_bounds__(kLossBlock) void k_splat_tile(SplatGeom g, const int* cell, const float* frac,
                                                           const float* target, float* image, float* resid,
                                                           float* partial) {
  static_assert(kImgTile * kImgTile == 64, "a lane per pixel, the wavefronts share the nodes");
  constexpr int kParts = kLossBlock / 64;
  __shared__ vf2 s_node[kSplatChunk];
  __shared__ int s_n;
  __shared__ long long s_acc[kLossBlock];
  const int ntx = (g.W + kImgTile - 1) / kImgTile;
  const int tid = threadIdx.x, lane = tid & 63;
  const int a0 = ((int)blockIdx.x % ntx) * kImgTile, b0 = ((int)blockIdx.x / ntx) * kImgTile;
  const int a = a0 + lane % kImgTile, b = b0 + lane / kImgTile;
  const bool live = a < g.W && b < g.H;
  const float px = -0.5f + ((float)a + 0.5f) * g.hx, py = -0.5f + ((float)b + 0.5f) * g.hy;
  // nodes farther from the tile's centre than its half side plus the cutoff
  // cannot reach a pixel centre of it (half a pixel and 0.1% of slack)
  const float mx = -0.5f + ((float)a0 + 0.5f * kImgTile) * g.hx, my = -0.5f + ((float)b0 + 0.5f * kImgTile) * g.hy;
  const float reach_x = 0.5f * kImgTile * g.hx + g.reach, reach_y = 0.5f * kImgTile * g.hy + g.reach;
  const float fnx = (float)g.nx, fny = (float)g.ny;
  long long acc = 0;
  for (int c0 = 0; c0 < g.n; c0 += kSplatChunk) {
    if (tid == 0) s_n = 0;
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kSplatChunk / kLossBlock; ++q) {
      const int i = c0 + q * kLossBlock + tid;
      float xw = 0.f, yw = 0.f;
      bool keep = false;
      if (i < g.n) {
        node_position(g, cell, frac, i, &xw, &yw);
        // (a tile that runs past the image lies up to one period further on)
        keep = fabsf(wrap_half(xw - mx, fnx)) <= reach_x && fabsf(wrap_half(yw - my, fny)) <= reach_y;
      }
      const unsigned long long m = __ballot(keep);
      if (m) {
        int base = 0;
        if (lane == 0) base = atomicAdd(&s_n, __popcll(m));
        base = __shfl(base, 0);
        const vf2 v = {xw, yw};
        if (keep) s_node[base + __popcll(m & ((1ull << lane) - 1ull))] = v;
      }
    }
    __syncthreads();
    const int n = s_n;
    for (int k = tid >> 6; k < n; k += kParts) {
      const vf2 v = s_node[k];
      const float dx = wrap_half(v.x - px, fnx), dy = wrap_half(v.y - py, fny);
      const float r2 = dx * dx + dy * dy;
      if (r2 <= g.cut2) acc += f32_to_fix(g.amp * expf(-r2 * g.inv2s2) * kImgFix);
    }
    __syncthreads();                              // the list is read before the next chunk
  }
  s_acc[tid] = acc;
  __syncthreads();
  if (tid >= 64) return;
#pragma unroll
  for (int q = 1; q < kParts; ++q) acc += s_acc[lane + 64 * q];
  float e2 = 0.f;
  if (live) {
    const int p = b * g.W + a;
    const float I = (float)((double)acc * kImgFixInv);
    const float r = I - target[p];
    if (image) image[p] = I;
    resid[p] = 2.0f * r / (float)(g.W * g.H);
    e2 = r * r;
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) e2 += __shfl_xor(e2, off);   // fixed pairing: deterministic
  if (lane == 0) partial[blockIdx.x] = e2;
}

// dL/dx, LANES lanes per node (a lane takes every LANES-th pixel of the node's
// window, the lanes' sums are joined by a fixed tree of shuffles).  The last
// block forms the loss.
template <int LANES>
__global__ __launch_bounds__(kLossBlock) void k_splat_grad(SplatGeom g, const int* cell, const float* frac,
                                                           const float* resid, float* g_pos, const float* partial,
                                                           int nblocks, float* loss) {
  if (blockIdx.x == gridDim.x - 1) {
    __shared__ double s_sum[kLossBlock];
    double acc = 0.0;
    for (int k = threadIdx.x; k < nblocks; k += kLossBlock) acc += (double)partial[k];
    s_sum[threadIdx.x] = acc;
    __syncthreads();
    for (int off = kLossBlock / 2; off > 0; off >>= 1) {
      if ((int)threadIdx.x < off) s_sum[threadIdx.x] += s_sum[threadIdx.x + off];
      __syncthreads();
    }
    if (threadIdx.x == 0) *loss = (float)(s_sum[0] / (double)(g.W * g.H));
    return;
  }
  const int per = kLossBlock / LANES, sub = threadIdx.x % LANES;
  for (int i = blockIdx.x * per + threadIdx.x / LANES; i < g.n; i += (gridDim.x - 1) * per) {
    float xw, yw;
    node_position(g, cell, frac, i, &xw, &yw);
    float gx = 0.f, gy = 0.f;
    for_node_pixels<LANES>(g, xw, yw, sub, [&](int pix, float dx, float dy, float v) {
      const float c = resid[pix] * v * g.inv_s2;
      gx -= c * dx;
      gy -= c * dy;
    });
#pragma unroll
    for (int off = LANES / 2; off > 0; off >>= 1) {
      gx += __shfl_xor(gx, off);
      gy += __shfl_xor(gy, off);
    }
    if (sub == 0) {
      g_pos[i] = gx;
      g_pos[g.n + i] = gy;
    }
  }
}

// Workspace: accumulator [H*W] u64 | residual [H*W] f32 | block sums (tile by
// tile they take the place of the accumulator, at most one per pixel).
size_t density_loss_workspace(int W, int H) {
  const size_t P = (size_t)W * H;
  const size_t nb = (P + kLossBlock - 1) / kLossBlock;
  auto al = [](size_t b) { return (b + 255) / 256 * 256; };
  return al(P * 8) + al(P * 4) + al(nb * 4);
}

void launch_density_loss(int nx, int ny, int n, int W, int H, float sigma, float amp, const int* cell,
                         const float* frac, const float* target, float* image, float* loss, float* g_pos,
                         void* ws, hipStream_t s) {
  SplatGeom g;
  g.nx = nx;
  g.ny = ny;
  g.n = n;
  g.W = W;
  g.H = H;
  g.hx = (float)nx / (float)W;
  g.hy = (float)ny / (float)H;
  g.inv2s2 = 1.0f / (2.0f * sigma * sigma);
  g.inv_s2 = 1.0f / (sigma * sigma);
  g.cut2 = 25.0f * sigma * sigma;
  g.reach = 5.005f * sigma;
  g.amp = amp;
  // a pixel k columns away from the node's own has its centre at least
  // (|k| - 1/2) hx away: columns up to 5 sigma / hx + 1/2 can be inside
  // (compared in floating point: half-widths past the integers' range too)
  const float rx = floorf(5.0f * sigma / g.hx + 0.5f) + 1.0f, ry = floorf(5.0f * sigma / g.hy + 0.5f) + 1.0f;
  g.rx = 2.0f * rx + 1.0f >= (float)W ? -1 : (int)rx;   // the window would wrap onto itself: all columns once
  g.ry = 2.0f * ry + 1.0f >= (float)H ? -1 : (int)ry;
  const int P = W * H;
  const int nb = (P + kLossBlock - 1) / kLossBlock;
  char* base = (char*)ws;
  auto al = [](size_t b) { return (b + 255) / 256 * 256; };
  unsigned long long* acc = (unsigned long long*)base;
  float* resid = (float*)(base + al((size_t)P * 8));
  float* partial = (float*)(base + al((size_t)P * 8) + al((size_t)P * 4));
  // How the image is summed, from the two ways' measured times in us over 100
  // to 262,144 nodes, 64^2 to 1024^2 pixels and windows of 25 to 2800 pixels:
  // tile by tile every block tests every node (3.2 us per 1000 nodes and 1024
  // blocks, 1.7 us per 1024 blocks besides); node by node costs two launches
  // more (6 us) and one HBM atomic per contribution (8 us per million).  1000
  // nodes on 128^2 pixels: 9.4 against 16.1 us; 8000 nodes: 33 against 15.8;
  // 65,536 nodes with windows of 2800 pixels: 478 against 1261.
  const int tiles = ((W + kImgTile - 1) / kImgTile) * ((H + kImgTile - 1) / kImgTile);
  const double wx = g.rx < 0 ? W : 2 * g.rx + 1, wy = g.ry < 0 ? H : 2 * g.ry + 1, win = wx * wy;
  const double covered = std::min((double)P, 3.1416 * (double)g.cut2 / ((double)g.hx * (double)g.hy));
  const bool by_tile = 3.2e-3 * n * std::max(1.0, tiles / 1024.0) + 1.7e-3 * tiles < 6.0 + 8e-6 * n * covered;
  const int thread_blocks = n / 256 + 1 < 4096 ? n / 256 + 1 : 4096;   // a thread per node
  const int wave_blocks = (n + 3) / 4;                                   // a wavefront per node
  if (by_tile) {
    partial = (float*)acc;
    k_splat_tile<<<tiles, kLossBlock, 0, s>>>(g, cell, frac, target, image, resid, partial);
  } else {
    const int zb = P / 256 + 1 < 1024 ? P / 256 + 1 : 1024;
    k_zero_u64<<<zb, 256, 0, s>>>(acc, P);
    // small windows leave most of a wavefront idle (25 pixels, 65,536 nodes:
    // 16.2 us by threads, 28.6 by wavefronts); larger ones make a thread's
    // loop long (121 pixels: 287 against 63 us)
    if (n == 0)
      ;                                          // (no block of wavefronts: the image is the cleared accumulator)
    else if (win <= 32)
      k_splat_image<1><<<thread_blocks, kLossBlock, 0, s>>>(g, cell, frac, acc);
    else
      k_splat_image<64><<<wave_blocks, kLossBlock, 0, s>>>(g, cell, frac, acc);
    k_image_residual<<<nb, kLossBlock, 0, s>>>(g, acc, target, image, resid, partial);
  }
  const int np = by_tile ? tiles : nb;
  // the gradient: a wavefront per node costs 0.3 ns per node and 64 pixels, a
  // thread per node 0.4 us per pixel of its loop until the chip is full (1000
  // nodes, 121 pixels: 1.4 against 58 us; 262,144 nodes: 129 against 73)
  const bool by_wave = 3e-4 * n * std::ceil(win / 64.0) < 0.4 * win * std::max(1.0, n / 262144.0);
  if (!g_pos || n == 0)
    k_splat_grad<1><<<1, kLossBlock, 0, s>>>(g, cell, frac, resid, g_pos, partial, np, loss);   // the loss alone
  else if (by_wave)
    k_splat_grad<64><<<wave_blocks + 1, kLossBlock, 0, s>>>(g, cell, frac, resid, g_pos, partial, np, loss);
  else
    k_splat_grad<1><<<thread_blocks + 1, kLossBlock, 0, s>>>(g, cell, frac, resid, g_pos, partial, np, loss);
}

// ---------------------------------------------------------------------------
// Efforts: per filament, sum over its joints of (old - new rest angle)^2 and
// over its edges of (old - new rest length)^2, accumulated into effort[f]
// and effort[F + f].  One block per filament; fixed-order block sums.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_rest_effort(int n_fil, const int* fil_offset, const int* fil_flags,
                                                     const float* old_a, const float* new_a, const float* old_l,
                                                     const float* new_l, float* effort) {
  __shared__ float s_b[256];
  __shared__ float s_p[256];
  for (int f = blockIdx.x; f < n_fil; f += gridDim.x) {
    const int a = fil_offset[f], b = fil_offset[f + 1], n = b - a;
    const bool ring = fil_flags && (fil_flags[f] & 1) && n >= 3;
    const int j0 = ring ? a : a + 1, j1 = ring ? b : b - 1;      // joints [j0, j1)
    const int e1 = ring ? b : b - 1;                               // edges [a, e1)
    float eb = 0.f, ep = 0.f;
    for (int i = j0 + (int)threadIdx.x; i < j1; i += 256) {
      const float d = old_a[i] - new_a[i];
      eb += d * d;
    }
    for (int i = a + (int)threadIdx.x; i < e1; i += 256) {
      const float d = old_l[i] - new_l[i];
      ep += d * d;
    }
    s_b[threadIdx.x] = eb;
    s_p[threadIdx.x] = ep;
    __syncthreads();
    for (int off = 128; off > 0; off >>= 1) {
      if ((int)threadIdx.x < off) {
        s_b[threadIdx.x] += s_b[threadIdx.x + off];
        s_p[threadIdx.x] += s_p[threadIdx.x + off];
      }
      __syncthreads();
    }
    if (threadIdx.x == 0) {
      effort[f] += s_b[0];
      effort[n_fil + f] += s_p[0];
    }
    __syncthreads();
  }
}

void launch_rest_effort(int n_fil, const int* fil_offset, const int* fil_flags, const float* old_a,
                        const float* new_a, const float* old_l, const float* new_l, float* effort, hipStream_t s) {
  if (n_fil <= 0) return;
  k_rest_effort<<<n_fil < 8192 ? n_fil : 8192, 256, 0, s>>>(n_fil, fil_offset, fil_flags, old_a, new_a, old_l, new_l,
                                                           effort);
}

}  // namespace mc
