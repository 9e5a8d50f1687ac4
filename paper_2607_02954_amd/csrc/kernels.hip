// Forward kernels of the filament-fluid step for gfx950 (CDNA4).
//
// Step order (all worlds of a table at once):
//   k_prepare     binned worlds: S0 actuation + S1 PBD Cosserat projection
//                 (Eqs. 1-4) -> node elastic force, beside S2 deposit + S3
//                 separable circular Gaussian filter on a tile with an
//                 (R+1)-cell halo, all in LDS, which writes the central
//                 difference G = D s~ of the filtered density
//                 (k_elastic and k_filter: the two alone)
//   k_repulse     S4 repulsion -k_rep sum W G -> total node force (sorted
//                 and direct transfers)
//   k_spread      S5 force spread onto a tile, summed in LDS; for the
//                 binned transfer it also forms S4 for the nodes it spreads
//   k_lbm         S6 D2Q9 TRT/Guo collision and push streaming over
//                 contiguous cells; exports u
//   k_integrate   S7 gather u at the nodes and move them; appends every node
//                 to the tile lists of the next step (binned transfer)
//   k_fluid_tile  S4 - S7 of binned worlds of few tiles in one kernel
//
// Particle -> grid transfer has three modes, chosen per world:
//   binned  every grid tile has a list of the nodes it needs (its own and those
//           around it) and sums their contributions in
//           LDS as 64-bit fixed point (integer adds: order-independent, so
//           results are bitwise reproducible, and on this chip integer LDS
//           atomics are far faster than float ones), then writes every cell
//           once: no HBM atomics and no clearing pass
//   sorted  nodes are counting-sorted by home cell and every grid value is a
//           fixed-order sum over the sorted segments of its 4x4 home window:
//           bitwise reproducible
//   direct  global float atomics into HBM accumulators (reference point)
//
// Node kernels run one block per node pack (whole filaments, <= pack nodes,
// filament-contiguous SoA), so neighbour exchange along a chain stays in LDS.
// Positions are an integer cell plus a float fraction, so the quantities the
// physics needs (edge vectors, kernel offsets) are formed from small numbers.
#include <hip/hip_ext.h>

#include <algorithm>

#include "device_util.h"

namespace mc {

// ---------------------------------------------------------------------------
// S0 + S1: actuation and PBD elastic force.  Then, by transfer mode: the
// home-cell key and rank (sorted) or the density deposit with global atomics
// (direct).
// ---------------------------------------------------------------------------
// Two-layer marker displacement of node gi (markers at x +- d): offset times
// the unit normal of the tangent x_b - x_a, a and b its neighbours (or the node
// itself at a chain end; zero for a lone node).
static __device__ __forceinline__ void marker_displacement(const WorldDev& w, int gi, int a, int b) {
  const int N = w.n_part;
  const MC_GLOBAL int* cell = glb(w.cell_in);
  const MC_GLOBAL float* frac = glb(w.frac_in);
  const float tx = (float)(cell[b] - cell[a]) + (frac[b] - frac[a]);
  const float ty = (float)(cell[N + b] - cell[N + a]) + (frac[N + b] - frac[N + a]);
  const float len = sqrtf(tx * tx + ty * ty);
  const float sc = len > 0.f ? w.marker_offset / len : 0.f;
  glb(w.d_marker)[gi] = -ty * sc;
  glb(w.d_marker)[N + gi] = tx * sc;
}

// GEN: worlds may pass closed-loop flags and per-edge stiffness arrays, BR
// (with GEN) branches as well; the plain variant serves open chains with the
// world's scalar stiffnesses.
//
// Branches: the first node c0 of a filament that hangs from node p (of the
// same pack: packs hold whole creatures) owns the attachment edge p -> c0,
// whose angle lives in s_ta at c0's slot, and its two joints; after the
// regular colours of each pass come the joints at the parent nodes, then
// those at the first nodes (bending), and the attachment edges (position).
// A node carries at most one attachment, so each of those phases touches
// every angle and node once at most.
template <int PACK, bool BR>
struct ElasticLds {
  float th[PACK];
  float dx[PACK];
  float dy[PACK];
  float ta[BR ? PACK : 1];
  int off[PACK + 1];
};

template <int PACK, bool GEN, bool BR>
static __device__ __forceinline__ void elastic_pack(const WorldDev& w, const Pack& pk, const Ctl& ctl,
                                                    ElasticLds<PACK, BR>& lds) {
  static_assert(GEN || !BR, "branches take the general variant");
  float* s_th = lds.th;
  float* s_dx = lds.dx;
  float* s_dy = lds.dy;
  float* s_ta = lds.ta;
  int* s_off = lds.off;
  const int li = threadIdx.x;
  {
    const int N = w.n_part, nx = w.nx, ny = w.ny, mode = w.mode;
    const MC_GLOBAL int* cell = glb(w.cell_in);
    const MC_GLOBAL float* frac = glb(w.frac_in);
    const MC_GLOBAL int* foff = glb(w.fil_offset);
    const int nf = pk.fil_end - pk.fil_begin;
    // every load this node needs is issued before anything waits: the
    // filament offsets first (they go to LDS), then the node's own data at
    // clamped indices (lanes past the pack's end, and the pack's last node
    // for its successor, read an in-range node and ignore it)
    const int off_a = foff[pk.fil_begin + min(li, nf)];      // nf <= PACK filaments
    const int off_b = foff[pk.fil_begin + nf];
    __builtin_amdgcn_sched_barrier(0);           // keep these two loads ahead of the node loads
    const int gi = pk.node_begin + li;
    const bool active = gi < pk.node_end;
    const int gic = min(gi, pk.node_end - 1);
    const int gin = min(gic + 1, N - 1);
    const int c0x = cell[gic], c0y = cell[N + gic];
    const float f0x = frac[gic], f0y = frac[N + gic];
    int c1x = cell[gin], c1y = cell[N + gin];
    float f1x = frac[gin], f1y = frac[N + gin];
    const float L_r = glb(w.rest_length)[gic];
    const float ra = glb(w.rest_angle)[gic];
    // per-edge stiffnesses (joint and edge at this node), else the world's
    const float kb_i = GEN && w.kb_arr ? glb(w.kb_arr)[gic] : w.k_bend;
    const float ks_i = GEN && w.ks_arr ? glb(w.ks_arr)[gic] : w.k_stretch;
    const float ksh_i = GEN && w.ksh_arr ? glb(w.ksh_arr)[gic] : w.k_shear;
    if (li < nf) s_off[li] = off_a - pk.node_begin;
    if (li == 0) s_off[nf] = off_b - pk.node_begin;
    __syncthreads();

    // filament of this node: largest f with s_off[f] <= li
    int lo = 0, hi = nf - 1;
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (s_off[mid] <= li) lo = mid; else hi = mid - 1;
    }
    const int o = s_off[lo];
    const int n = s_off[lo + 1] - o;
    const int k = li - o;
    const int fil = pk.fil_begin + lo;
    // a closed loop (at least three nodes): the last node's edge joins it to
    // the first, and every node is a joint (the first between the closing
    // edge and edge 0)
    const bool ring = GEN && w.fil_flags && (glb(w.fil_flags)[fil] & 1) && n >= 3;
    const bool has_edge = active && (k < n - 1 || ring);
    const bool is_joint = active && (ring || (k >= 1 && k <= n - 2));
    const int j = ring ? k : k - 1;              // joint's local index
    const int m = ring ? n : n - 2;              // joints of the filament
    const int li_prev = (ring && k == 0) ? o + n - 1 : li - 1;    // edge before the joint
    const int li_next = (ring && k == n - 1) ? o : li + 1;        // far node of the edge
    if (ring && k == n - 1) {                    // the closing edge's far node: the first
      const int g0 = pk.node_begin + o;
      c1x = cell[g0];
      c1y = cell[N + g0];
      f1x = frac[g0];
      f1y = frac[N + g0];
    }
    // Gauss-Seidel colours: local parity; on a loop of odd length the last
    // joint and the last edge meet the first ones and take a third colour
    const int jcol = (ring && (n & 1) && j == n - 1) ? 2 : (j & 1);
    const int ecol = (ring && (n & 1) && k == n - 1) ? 2 : (k & 1);
    int ncol = 2;                                // block-uniform
    if constexpr (GEN) ncol = __syncthreads_or(active && ring && (n & 1)) ? 3 : 2;
    const float amp = glb(w.act_amp)[fil], period = glb(w.act_period)[fil], phase = glb(w.act_phase)[fil];

    const int cx = active ? c0x : 0, cy = active ? c0y : 0;
    const float fx = active ? f0x : 0.f, fy = active ? f0y : 0.f;
    float v0x = 0.f, v0y = 0.f, L = 0.f, th = 0.f;
    float u0x = 1.f, u0y = 0.f;                  // unit edge direction, (cos th, sin th)
    if (has_edge) {
      v0x = (float)(c1x - cx) + (f1x - fx);
      v0y = (float)(c1y - cy) + (f1y - fy);
      L = L_r;
      th = atan2f(v0y, v0x);
      const float l0 = hw_sqrt(v0x * v0x + v0y * v0y);
      if (l0 > 0.f) {
        const float il = hw_rcp(l0);
        u0x = v0x * il;
        u0y = v0y * il;
      }
    }
    float th_hat = 0.f;
    if (is_joint) th_hat = actuated_angle(ra, amp, period, phase, ctl.t, j, m);
    s_th[li] = th;
    s_dx[li] = 0.f;
    s_dy[li] = 0.f;
    // branch attachment owned by this node (its filament's first node)
    bool att = false, att_cj = false, any_att = false;
    int p_l = 0, in_l = 0;
    float a_vx = 0.f, a_vy = 0.f, a_th = 0.f, a_ux = 1.f, a_uy = 0.f, a_L = 0.f, a_al = 0.f, a_be = 0.f;
    if (BR && w.fil_parent) {                    // block-uniform: the pack's world
      const int par = (active && k == 0) ? glb(w.fil_parent)[fil] : -1;
      att = par >= 0;
      if (att) {
        p_l = par - pk.node_begin;
        int lp = 0, hp = nf - 1;                   // p's filament: largest f with s_off[f] <= p_l
        while (lp < hp) {
          const int mid = (lp + hp + 1) >> 1;
          if (s_off[mid] <= p_l) lp = mid; else hp = mid - 1;
        }
        in_l = p_l == s_off[lp] ? s_off[lp + 1] - 1 : p_l - 1;   // p's entering edge
        const int F = w.n_fil;
        a_L = glb(w.fil_attach)[fil];
        a_al = glb(w.fil_attach)[F + fil];
        a_be = glb(w.fil_attach)[2 * F + fil];
        a_vx = (float)(cx - cell[par]) + (fx - frac[par]);
        a_vy = (float)(cy - cell[N + par]) + (fy - frac[N + par]);
        a_th = atan2f(a_vy, a_vx);
        const float l0 = hw_sqrt(a_vx * a_vx + a_vy * a_vy);
        if (l0 > 0.f) {
          const float il = hw_rcp(l0);
          a_ux = a_vx * il;
          a_uy = a_vy * il;
        }
        att_cj = n >= 2;
      }
      s_ta[li] = a_th;
      any_att = __syncthreads_or(att);
    }
    __syncthreads();
    const float hb_w = 0.5f * w.k_bend, hs_w = 0.5f * w.k_stretch, ksh_w = w.k_shear;

    const float hb = 0.5f * kb_i;
    const float hs = 0.5f * ks_i;
    const float ksh = ksh_i;
    const int iters = w.pbd_iters;
    for (int iter = 0; iter < iters; ++iter) {
      // bending pass (Eq. 1): even joints, then odd joints (then a loop's third colour)
      for (int par = 0; par < ncol; ++par) {
        if (is_joint && jcol == par) {
          const float t1 = s_th[li_prev];
          const float t2 = s_th[li];
          const float c = wrap_angle(t2 - t1) - th_hat;
          s_th[li_prev] = t1 + hb * c;
          s_th[li] = t2 - hb * c;
        }
        __syncthreads();
      }
      if (BR && any_att) {                       // attachment joints: at p, then at c0
        if (att) {
          const float t1 = s_th[in_l], t2 = s_ta[li];
          const float c = wrap_angle(t2 - t1) - a_al;
          s_th[in_l] = t1 + hb_w * c;
          s_ta[li] = t2 - hb_w * c;
        }
        __syncthreads();
        if (att_cj) {
          const float t1 = s_ta[li], t2 = s_th[li];
          const float c = wrap_angle(t2 - t1) - a_be;
          s_ta[li] = t1 + hb_w * c;
          s_th[li] = t2 - hb_w * c;
        }
        __syncthreads();
      }
      // the edge directions of this iteration (the angles change only in the
      // bending passes), for every lane at once rather than per colour
      float cs = 1.f, sn = 0.f;
      if (has_edge) edge_direction(s_th[li], th, u0x, u0y, &cs, &sn);
      float a_cs = 1.f, a_sn = 0.f;
      if (BR && att) edge_direction(s_ta[li], a_th, a_ux, a_uy, &a_cs, &a_sn);
      // position pass (Eqs. 2-4): even edges, then odd edges (then the third colour)
      for (int par = 0; par < ncol; ++par) {
        if (has_edge && ecol == par) {
          const float d0x = s_dx[li], d0y = s_dy[li];
          const float d1x = s_dx[li_next], d1y = s_dy[li_next];
          const float vx = v0x + (d1x - d0x);
          const float vy = v0y + (d1y - d0y);
          const float ell = hw_sqrt(vx * vx + vy * vy);
          const float sc = (ell - L) * hw_rcp(ell);
          const float csx = sc * vx, csy = sc * vy;
          const float dx = hs * (csx + ksh * (vx - L * cs - csx));
          const float dy = hs * (csy + ksh * (vy - L * sn - csy));
          s_dx[li] = d0x + dx;
          s_dy[li] = d0y + dy;
          s_dx[li_next] = d1x - dx;
          s_dy[li_next] = d1y - dy;
        }
        __syncthreads();
      }
      if (BR && any_att) {                       // attachment edges p -> c0
        if (att) {
          const float d0x = s_dx[p_l], d0y = s_dy[p_l];
          const float d1x = s_dx[li], d1y = s_dy[li];
          const float vx = a_vx + (d1x - d0x);
          const float vy = a_vy + (d1y - d0y);
          const float ell = hw_sqrt(vx * vx + vy * vy);
          const float sc = (ell - a_L) * hw_rcp(ell);
          const float csx = sc * vx, csy = sc * vy;
          const float dx = hs_w * (csx + ksh_w * (vx - a_L * a_cs - csx));
          const float dy = hs_w * (csy + ksh_w * (vy - a_L * a_sn - csy));
          s_dx[p_l] = d0x + dx;
          s_dy[p_l] = d0y + dy;
          s_dx[li] = d1x - dx;
          s_dy[li] = d1y - dy;
        }
        __syncthreads();
      }
    }

    const int bx = wrap_index(cx, nx);
    const int by = wrap_index(cy, ny);
    if (active) {
      MC_GLOBAL float* fel = glb(w.fel_el);
      fel[gi] = w.k_el * s_dx[li];
      fel[N + gi] = w.k_el * s_dy[li];
    }
    if (w.d_marker) {                            // block-uniform: two-layer markers of the pack
      const int before = k > 0 ? li - 1 : (ring ? o + n - 1 : li);
      const int after = k < n - 1 ? li + 1 : (ring ? o : li);
      if (active) marker_displacement(w, gi, pk.node_begin + before, pk.node_begin + after);
    }
    if (mode == kSorted) {
      if (active) {
        const int key = by * nx + bx;
        glb(w.key)[gi] = key;
        glb(w.rank)[gi] = atomicAdd((int*)(glb(w.cnt) + key), 1);
      }
    } else if (active && mode == kDirect) {
      float wx[4], wy[4];
      peskin4(fx, wx);
      peskin4(fy, wy);
      int ix[4];
#pragma unroll
      for (int a = 0; a < 4; ++a) ix[a] = wrap_near(bx - 1 + a, nx);
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        MC_GLOBAL float* row = glb(w.s) + (size_t)wrap_near(by - 1 + b, ny) * nx;
#pragma unroll
        for (int a = 0; a < 4; ++a) unsafeAtomicAdd((float*)(row + ix[a]), wx[a] * wy[b]);
      }
    }
  }
}

template <int PACK, bool GEN, bool BR>
__global__ __launch_bounds__(PACK) void k_elastic(const WorldDev* __restrict__ W, Tables T) {
  __shared__ ElasticLds<PACK, BR> lds;
  const int npk = *T.n_packs;
  for (int it = blockIdx.x; it < npk; it += gridDim.x) {
    const Pack pk = T.packs[it];
    const WorldDev& w = W[pk.world];
    const Ctl ctl = *w.ctl_src;
    if (ctl.remaining <= 0) continue;           // block-uniform
    elastic_pack<PACK, GEN, BR>(w, pk, ctl, lds);
    __syncthreads();
  }
}


// ---------------------------------------------------------------------------
// Binned transfer, pre-pass of a run: the tile lists of the current positions
// (each step's integration then appends the next step's).  Own nodes that their
// tile's segment does not hold are counted by the pass that writes the others;
// a pass over the tiles then hands out the spill area, and a last one over the
// nodes fills it (both end at once where there are none, 9 us for 1,048,576 nodes
// on 2048^2 in place of 24, and leave the near and far nodes that overflowed to
// the tiles around for one step).
// ---------------------------------------------------------------------------
// Empty lists; and with n_steps >= 0 the control words of a run of that many
// steps from step t (one launch rather than one more per world).
__global__ __launch_bounds__(256) void k_lists_zero(const WorldDev* __restrict__ W, Tables T, long long t, int n_steps) {
  for (int k = blockIdx.y; k < *T.n_worlds; k += gridDim.y) {
    const WorldDev& w = W[T.worlds[k].x];
    if (n_steps >= 0 && blockIdx.x == 0 && threadIdx.x == 0) {
      Ctl c;
      c.t = t;
      c.remaining = n_steps;
      c.pad = 0;
      *(Ctl*)w.ctl_src = c;
    }
    if (w.mode != kBinned || w.tl_kind == kNoLists || (n_steps >= 0 ? n_steps : w.ctl_src->remaining) <= 0) continue;
    const int nt = w.ntx * w.nty, n = nt * kListCounts + kListWords;
    for (int i = blockIdx.x * 256 + threadIdx.x; i < n; i += gridDim.x * 256) {
      const int tile = i / kListCounts, seg = i - tile * kListCounts - kFirst;
      glb(w.tl_cnt)[i] = tile < nt && seg >= 0 && seg < kSegs ? tile * w.tl_stride + segment_first(w, seg) : 0;
    }
  }
}

// The world's words after its tiles' counts.
static __device__ __forceinline__ MC_GLOBAL int* list_words(const WorldDev& w, MC_GLOBAL int* counts) {
  return counts + w.ntx * w.nty * kListCounts;
}

// Flags of the lists that cannot be used when segment seg of tile (tx, ty)'s
// list is full.
static __device__ __forceinline__ void flag_overflow(const WorldDev& w, MC_GLOBAL int* counts, int tx, int ty, int seg) {
  if (seg != kCntOwn) {
    atomicOr((int*)(counts + (ty * w.ntx + tx) * kListCounts + kCntFlags),
             seg == kCntStrays ? kOverStrays : kOverSegment);
    return;
  }
  const int mx = min(w.ntx, 5), my = min(w.nty, 5);   // the tiles that may have to read these own nodes
#pragma unroll 1
  for (int k = 0; k < mx * my; ++k) {
    const int j = k / mx, i = k - j * mx;
    const int t = (w.nty <= 5 ? j : wrap_near(ty - 2 + j, w.nty)) * w.ntx + (w.ntx <= 5 ? i : wrap_near(tx - 2 + i, w.ntx));
    atomicOr((int*)(counts + t * kListCounts + kCntFlags), kOverOwn);
  }
}

// Entry e of the own nodes: their record, or their index alone.
static __device__ __forceinline__ void write_entry(const WorldDev& w, MC_GLOBAL vi4* lists, int e, const vi4& rec) {
  if (w.tl_kind == kOwnIndices) ((MC_GLOBAL int*)lists)[e] = rec.w;
  else lists[e] = rec;
}

// Segment of neighbour q's nodes of class 1 (near) or 2 (far).
static __device__ __forceinline__ int class_segment(int cls, int q) {
  return kCntNear - 8 + 8 * cls + q;
}

static __device__ __forceinline__ void append_stray(const WorldDev& w, MC_GLOBAL vi4* lists, MC_GLOBAL int* counts,
                                                    int tx, int ty, const vi4& rec) {
  const int tile = ty * w.ntx + tx;
  const int k = atomicAdd((int*)(counts + tile * kListCounts + kCntStrays), 1);
  if (k < w.tl_strays) lists[(size_t)tile * w.tl_stride + w.tl_strays - 1 - k] = rec;
  else flag_overflow(w, counts, tx, ty, kCntStrays);
}
// The record as a stray of every tile it reaches beyond the 3x3 around (cx, cy).
template <int TILE>
static __device__ __forceinline__ void append_strays(const WorldDev& w, MC_GLOBAL vi4* lists, MC_GLOBAL int* counts,
                                                     int cx, int cy, const vi4& rec) {
  for_reached_tiles<TILE>(w, rec.x & 0xffff, rec.x >> 16, [&](int tx, int ty, int) {
    if (next_to(w, cx, cy, tx, ty)) return;
    append_stray(w, lists, counts, tx, ty, rec);
  });
}

// Node gi into the segments of the lists it belongs to: the first pass counts
// all and writes what its place in the list holds (and the strays), the second
// (SPILL) fills the segments that lie in the spill area.  last: no second one follows.
template <int TILE, bool SPILL>
static __device__ __forceinline__ void build_lists_of_node(const WorldDev& w, int gi, bool last) {
  constexpr int sh = TileCfg<TILE>::kShift;
  const vi4 rec = node_record(w, gi);
  const int hx = rec.x & 0xffff, hy = rec.x >> 16;
  const int cx = hx >> sh, cy = hy >> sh, ntx = w.ntx, nty = w.nty;
  const bool segments = w.tl_kind == kSegments;
  MC_GLOBAL vi4* lists = glbv<vi4>(w.tl_rec);
  MC_GLOBAL int* counts = glb(w.tl_cnt);
  const Classes c = neighbour_classes<TILE>(w, cx, cy, hx, hy);
  const Pairs a(c);
  const auto tile_at = [&](int dx, int dy) { return nb_tile(cy, dy, nty) * ntx + nb_tile(cx, dx, ntx); };
  const auto wanted = [&](int tile, int seg) {
    return !SPILL || counts[tile * kListCounts + kFirst + seg] >= ntx * nty * w.tl_stride;
  };
  const auto put = [&](int tile, int seg, int slot) {
    if (SPILL || slot < segment_cap(w, seg))
      write_entry(w, lists, (SPILL ? counts[tile * kListCounts + kFirst + seg] : tile * w.tl_stride + segment_first(w, seg)) + slot,
                  rec);
    else if (seg == kCntOwn && !last) list_words(w, counts)[kWordOver] = 1;
    else flag_overflow(w, counts, tile % ntx, tile / ntx, seg);
    if (!SPILL && seg != kCntOwn && slot >= segment_cap(w, seg)) counts[(cy * ntx + cx) * kListCounts + kCntCrowded] = 1;
  };
  // one atomic per list segment and wavefront, whose nodes share few tiles;
  // every one is issued before the first result is used (1,048,576 nodes:
  // 65.7 -> 32 us; 38 with the places of segments that may lie in the spill area)
  const int t0 = cy * ntx + cx, t1 = tile_at(a.dx, 0), t2 = tile_at(0, a.dy), t3 = tile_at(a.dx, a.dy);
  const int q1 = class_segment(a.side_x, a.qx()), q2 = class_segment(a.side_y, a.qy()), q3 = class_segment(a.corner, a.qc());
  const bool pairs = segments && !a.more;
  const bool h0 = wanted(t0, kCntOwn), h1 = pairs && a.side_x < 3 && wanted(t1, q1),
             h2 = pairs && a.side_y < 3 && wanted(t2, q2), h3 = pairs && a.corner < 3 && wanted(t3, q3);
  const int k0 = kListCounts * t0 + kCntOwn, k1 = kListCounts * t1 + q1, k2 = kListCounts * t2 + q2, k3 = kListCounts * t3 + q3;
  const AggGroup g0(k0, h0), g1(k1, h1), g2(k2, h2), g3(k3, h3);
  const int lane = __lane_id();
  int s0 = 0, s1 = 0, s2 = 0, s3 = 0;
  if (h0 && g0.leader == lane) s0 = atomicAdd((int*)(counts + k0), g0.count);
  if (h1 && g1.leader == lane) s1 = atomicAdd((int*)(counts + k1), g1.count);
  if (h2 && g2.leader == lane) s2 = atomicAdd((int*)(counts + k2), g2.count);
  if (h3 && g3.leader == lane) s3 = atomicAdd((int*)(counts + k3), g3.count);
  s0 = __shfl(s0, g0.leader) + g0.rank;
  s1 = __shfl(s1, g1.leader) + g1.rank;
  s2 = __shfl(s2, g2.leader) + g2.rank;
  s3 = __shfl(s3, g3.leader) + g3.rank;
  if (h0) put(t0, kCntOwn, s0);
  if (h1) put(t1, q1, s1);
  if (h2) put(t2, q2, s2);
  if (h3) put(t3, q3, s3);
  if (!segments || !a.more) return;
  int slot[8];
  static_for<8>([&](auto qq) {
    constexpr int q = decltype(qq)::value;
    const int t = tile_at(nb_dx(q), nb_dy(q)), seg = class_segment(c.of(q), q);
    slot[q] = -1;
    if (c.of(q) <= 2 && wanted(t, seg)) slot[q] = atomicAdd((int*)(counts + kListCounts * t + seg), 1);
  });
  static_for<8>([&](auto qq) {
    constexpr int q = decltype(qq)::value;
    if (slot[q] >= 0) put(tile_at(nb_dx(q), nb_dy(q)), class_segment(c.of(q), q), slot[q]);
  });
  if (!SPILL && c.beyond) append_strays<TILE>(w, lists, counts, cx, cy, rec);
}

// Room in the spill area for the segments that need it, where some tile's own
// nodes do; their nodes are counted again as they are written.
__global__ __launch_bounds__(256) void k_lists_reserve(const WorldDev* __restrict__ W, Tables T) {
  for (int k = blockIdx.y; k < *T.n_worlds; k += gridDim.y) {
    const WorldDev& w = W[T.worlds[k].x];
    if (w.mode != kBinned || w.tl_kind == kNoLists || w.ctl_src->remaining <= 0) continue;
    MC_GLOBAL int* counts = glb(w.tl_cnt);
    MC_GLOBAL int* words = list_words(w, counts);
    if (!words[kWordOver]) continue;
    const int nt = w.ntx * w.nty, segs = w.tl_kind == kSegments ? kSegs : 1;
    for (int t = blockIdx.x * 256 + threadIdx.x; t < nt; t += gridDim.x * 256) {
      MC_GLOBAL int* c = counts + t * kListCounts;
      const auto need = [&](int seg) { return seg == kCntStrays || c[seg] <= segment_cap(w, seg) ? 0 : c[seg]; };
      int n = 0;
      for (int seg = 0; seg < segs; ++seg) n += need(seg);
      if (n == 0) continue;
      int at = atomicAdd((int*)(words + kWordOwnSpill), n);
      bool all = true;
      for (int seg = 0; seg < segs; ++seg) {
        const int m = need(seg);
        if (m == 0) continue;
        if (at >= 0 && m <= w.tl_spill - at) {
          c[kFirst + seg] = nt * w.tl_stride + at;
          c[seg] = 0;
        } else {
          flag_overflow(w, counts, t % w.ntx, t / w.ntx, seg);
          all = false;
        }
        at += m;
      }
      if (all) atomicAnd((int*)(c + kCntFlags), ~kOverSegment);
    }
  }
}

template <int PACK, bool SPILL>
__global__ __launch_bounds__(PACK) void k_lists_build(const WorldDev* __restrict__ W, Tables T, int last) {
  const int npk = *T.n_packs;
  for (int it = blockIdx.x; it < npk; it += gridDim.x) {
    const Pack pk = T.packs[it];
    const WorldDev& w = W[pk.world];
    if (w.mode != kBinned || w.tl_kind == kNoLists || w.ctl_src->remaining <= 0) continue;
    if (SPILL && !list_words(w, glb(w.tl_cnt))[kWordOver]) continue;
    const int gi = pk.node_begin + threadIdx.x;
    if (gi >= pk.node_end) continue;
    if (w.tile_shift == 4) build_lists_of_node<16, SPILL>(w, gi, last);
    else build_lists_of_node<32, SPILL>(w, gi, last);
  }
}

// ---------------------------------------------------------------------------
// Sorted transfer: exclusive scan of the per-cell counts (three phases over
// (world, 1024-cell block) items), scatter of node indices into their slots,
// and an insertion sort of every multi-node segment by node index, so that
// all later sums run in a fixed order.
// ---------------------------------------------------------------------------
constexpr int kScanBlock = 1024;   // cells per scan item (256 threads x 4)

__global__ __launch_bounds__(256) void k_scan_reduce(const WorldDev* __restrict__ W, Tables T) {
  __shared__ int s_wave[4];
  const int n = *T.n_scan;
  for (int it = blockIdx.x; it < n; it += gridDim.x) {
    const int2 sc = T.scan[it];
    const WorldDev& w = W[sc.x];
    if (w.mode != kSorted || w.ctl_src->remaining <= 0) continue;
    const MC_GLOBAL int* cnt = glb(w.cnt);
    const int ncell = w.nx * w.ny;
    const int c0 = sc.y * kScanBlock + threadIdx.x * 4;
    int v = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) v += (c0 + k < ncell) ? cnt[c0 + k] : 0;
    int total;
    block_scan256(v, s_wave, &total);
    if (threadIdx.x == 0) glb(w.part)[sc.y] = total;
  }
}

__global__ __launch_bounds__(256) void k_scan_partials(const WorldDev* __restrict__ W, Tables T) {
  __shared__ int s_wave[4];
  const int n = *T.n_worlds;
  for (int it = blockIdx.x; it < n; it += gridDim.x) {
    const WorldDev& w = W[T.worlds[it].x];
    if (w.mode != kSorted || w.ctl_src->remaining <= 0) continue;
    MC_GLOBAL int* part = glb(w.part);
    const int ncell = w.nx * w.ny;
    const int nb = (ncell + kScanBlock - 1) / kScanBlock;
    int carry = 0;
    for (int b0 = 0; b0 < nb; b0 += 256) {
      const int b = b0 + threadIdx.x;
      const int v = b < nb ? part[b] : 0;
      int total;
      const int ex = block_scan256(v, s_wave, &total);
      if (b < nb) part[b] = carry + ex;
      carry += total;
    }
    if (threadIdx.x == 0) glb(w.start)[ncell] = carry;
  }
}

__global__ __launch_bounds__(256) void k_scan_down(const WorldDev* __restrict__ W, Tables T) {
  __shared__ int s_wave[4];
  const int n = *T.n_scan;
  for (int it = blockIdx.x; it < n; it += gridDim.x) {
    const int2 sc = T.scan[it];
    const WorldDev& w = W[sc.x];
    if (w.mode != kSorted || w.ctl_src->remaining <= 0) continue;
    MC_GLOBAL int* cnt = glb(w.cnt);
    MC_GLOBAL int* start = glb(w.start);
    const int ncell = w.nx * w.ny;
    const int c0 = sc.y * kScanBlock + threadIdx.x * 4;
    int v[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = (c0 + k < ncell) ? cnt[c0 + k] : 0;
    int total;
    const int ex = block_scan256(v[0] + v[1] + v[2] + v[3], s_wave, &total);
    int run = glb(w.part)[sc.y] + ex;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if (c0 + k < ncell) {
        start[c0 + k] = run;
        cnt[c0 + k] = 0;          // ready for the next step's histogram
      }
      run += v[k];
    }
  }
}

template <int PACK>
__global__ __launch_bounds__(PACK) void k_scatter(const WorldDev* __restrict__ W, Tables T) {
  const int npk = *T.n_packs;
  for (int it = blockIdx.x; it < npk; it += gridDim.x) {
    const Pack pk = T.packs[it];
    const WorldDev& w = W[pk.world];
    if (w.mode != kSorted || w.ctl_src->remaining <= 0) continue;
    const int gi = pk.node_begin + threadIdx.x;
    if (gi >= pk.node_end) continue;
    glb(w.perm)[glb(w.start)[glb(w.key)[gi]] + glb(w.rank)[gi]] = gi;
  }
}

template <int PACK>
__global__ __launch_bounds__(PACK) void k_segsort(const WorldDev* __restrict__ W, Tables T) {
  const int npk = *T.n_packs;
  for (int it = blockIdx.x; it < npk; it += gridDim.x) {
    const Pack pk = T.packs[it];
    const WorldDev& w = W[pk.world];
    if (w.mode != kSorted || w.ctl_src->remaining <= 0) continue;
    const int gi = pk.node_begin + threadIdx.x;
    // one thread per segment: the node that drew rank 0 (ranks are never rewritten)
    if (gi >= pk.node_end || glb(w.rank)[gi] != 0) continue;
    MC_GLOBAL int* perm = glb(w.perm);
    const int key = glb(w.key)[gi];
    const int b = glb(w.start)[key], e = glb(w.start)[key + 1];
    for (int i = b + 1; i < e; ++i) {
      const int v = perm[i];
      int j = i - 1;
      while (j >= b && perm[j] > v) {
        perm[j + 1] = perm[j];
        --j;
      }
      perm[j + 1] = v;
    }
    // fractions of the sorted nodes for the density gather of this step
    const int N = w.n_part;
    const MC_GLOBAL float* frac = glb(w.frac_in);
    MC_GLOBAL vf4* rec = glbv<vf4>(w.rec);
    for (int i = b; i < e; ++i) {
      const int v = perm[i];
      const vf4 r = {frac[v], frac[N + v], 0.f, 0.f};
      rec[i] = r;
    }
  }
}

// Fixed-order sums over the sorted segments of the 4x4 home window of cell
// (gx, gy): the node at home cell h contributes weight index c - h + 1.
__device__ __forceinline__ float gather_density(const MC_GLOBAL int* start, const MC_GLOBAL vf4* rec,
                                                int nx, int ny, int gx, int gy) {
  float acc = 0.f;
  for (int b = 0; b < 4; ++b) {
    const int hy = wrap_near(gy + 1 - b, ny);
    for (int a = 0; a < 4; ++a) {
      const int h = hy * nx + wrap_near(gx + 1 - a, nx);
      const int e = start[h + 1];
      for (int sidx = start[h]; sidx < e; ++sidx) {
        const vf4 r = rec[sidx];
        float wx[4], wy[4];
        peskin4(r.x, wx);
        peskin4(r.y, wy);
        acc += wx[a] * wy[b];
      }
    }
  }
  return acc;
}

__device__ __forceinline__ vf2 gather_force(const MC_GLOBAL int* start, const MC_GLOBAL vf4* rec,
                                               int nx, int ny, int gx, int gy) {
  float Fx = 0.f, Fy = 0.f;
  for (int b = 0; b < 4; ++b) {
    const int hy = wrap_near(gy + 1 - b, ny);
    for (int a = 0; a < 4; ++a) {
      const int h = hy * nx + wrap_near(gx + 1 - a, nx);
      const int e = start[h + 1];
      for (int sidx = start[h]; sidx < e; ++sidx) {
        const vf4 r = rec[sidx];
        float wx[4], wy[4];
        peskin4(r.x, wx);
        peskin4(r.y, wy);
        const float ww = wx[a] * wy[b];
        Fx += ww * r.z;
        Fy += ww * r.w;
      }
    }
  }
  const vf2 out = {Fx, Fy};
  return out;
}

// ---------------------------------------------------------------------------
// S2 + S3: density on a tile (side TILE) plus an (R+1)-cell halo, staged in LDS,
// the separable circular Gaussian (x pass, then y pass, both in LDS) on the
// tile plus a one-cell ring, and the central difference G = D s~ of the
// tile, written as interleaved float2.
//
// Binned mode deposits the neighbourhood's nodes into a padded window (three
// spare cells per side, see the window note with tile_spread_vec) as exact
// integer products of quantised weights, so the sums are order-independent
// and the inner loop is two 24-bit multiplies and an LDS add per cell.
// LDS: [window: filter_window_bytes(max radius) | density].
// ---------------------------------------------------------------------------
// Window rows are kWinPad elements longer than the window side: an even
// row length of 64-bit words puts vertically adjacent cells, which nodes
// next to each other on a chain often deposit to at once, in the same LDS bank.
constexpr int kWinPad = 1;
template <int TILE>
static __host__ __device__ constexpr int filter_window_bytes(int max_radius) {
  return (TILE + 2 + 2 * max_radius + 6) * (TILE + 2 + 2 * max_radius + 6 + kWinPad) * 8;
}
template <int TILE>
static __host__ __device__ constexpr int filter_density_bytes(int max_radius) {
  return (TILE + 2 + 2 * max_radius) * (TILE + 2 + 2 * max_radius) * 4;
}
// the passes' intermediate rows (region x ring) and the filtered ring fit the window
static_assert(filter_window_bytes<16>(1) >= ((16 + 2 + 2 * kMaxRadius) * 18 + 18 * 18) * 4, "window");
static_assert(filter_window_bytes<32>(1) >= ((32 + 2 + 2 * kMaxRadius) * 34 + 34 * 34) * 4, "window");
static_assert(filter_window_bytes<64>(1) >= ((64 + 2 + 2 * kMaxRadius) * 66 + 66 * 66) * 4, "window");

// q = k / d for 0 <= k < 2^16 and 0 < d <= 64: (k + 1/2) / d is at least
// 1/(2d) away from an integer, far beyond the FP32 rounding of the product.
static __device__ __forceinline__ int div_small(int k, float inv_d) {
  return (int)(((float)k + 0.5f) * inv_d);
}

// The two passes of the separable Gaussian (radius R) over the density
// region s_regf (reg x reg, reg = ring + 2R) into the filtered tile-plus-ring
// s_st (ring x ring, ring = TILE + 2), through s_mid (reg rows x ring).
// Every thread forms two adjacent outputs from taps read as aligned pairs
// (rows have even lengths); each output is summed in the same order as a
// one-output loop would.  Ends with a barrier.
template <int TILE, int NT, int R>
static __device__ __forceinline__ void filter_passes(const float* s_regf, float* s_mid, float* s_st, const float* g) {
  constexpr int kRing = TILE + 2, kThreads = NT;
  constexpr int reg = kRing + 2 * R, kHalf = kRing / 2;
  const int tid = threadIdx.x;
  for (int k = tid; k < reg * kHalf; k += kThreads) {
    const int r = k / kHalf, c = 2 * (k - (k / kHalf) * kHalf);
    const vf2* row = (const vf2*)(s_regf + r * reg + c);   // cells c .. c + 2R + 1 of row r
    float v[2 * R + 2];
#pragma unroll
    for (int i = 0; i <= R; ++i) {
      const vf2 t = row[i];
      v[2 * i] = t.x;
      v[2 * i + 1] = t.y;
    }
    float a0 = g[0] * v[R], a1 = g[0] * v[R + 1];
#pragma unroll
    for (int m = 1; m <= R; ++m) {
      a0 += g[m] * (v[R - m] + v[R + m]);
      a1 += g[m] * (v[R + 1 - m] + v[R + 1 + m]);
    }
    const vf2 out = {a0, a1};
    *(vf2*)(s_mid + r * kRing + c) = out;
  }
  __syncthreads();
  for (int k = tid; k < kRing * kHalf; k += kThreads) {
    const int r = k / kHalf, c = 2 * (k - (k / kHalf) * kHalf);
    const vf2* col = (const vf2*)(s_mid + (r + R) * kRing + c);
    vf2 t[2 * R + 1];
#pragma unroll
    for (int m = -R; m <= R; ++m) t[m + R] = col[m * kHalf];
    float a0 = g[0] * t[R].x, a1 = g[0] * t[R].y;
#pragma unroll
    for (int m = 1; m <= R; ++m) {
      a0 += g[m] * (t[R - m].x + t[R + m].x);
      a1 += g[m] * (t[R - m].y + t[R + m].y);
    }
    const vf2 out = {a0, a1};
    *(vf2*)(s_st + r * kRing + c) = out;
  }
  __syncthreads();
}

// Whether a segment with n nodes and room for cap may be outgrown by the next step.
static __device__ __forceinline__ bool nearly_full(int n, int cap) { return n + (n >> 3) + 4 > cap; }
// Places for the segments that the block of a tile will write in this step's
// integration where one may outgrow its place, in the spill area for those that may outgrow theirs: its own nodes
// and strays are all that it can come to integrate, of the others there will be
// about as many as now.  Left in the next lists, the capacities in place of the
// numbers.  (Here rather than in the integration, whose registers it would cost.)
static __device__ __forceinline__ void reserve_segments(const WorldDev& w, int bx, int by) {
  const int seg = threadIdx.x;
  if (seg >= kSegs || seg == kCntStrays) return;
  const bool own = seg == kCntOwn;
  const int q = (seg - kCntNear) & 7, dx = own ? 0 : nb_dx(q), dy = own ? 0 : nb_dy(q);
  if (!nb_exists(dx, w.ntx) || !nb_exists(dy, w.nty)) return;
  const int tile = nb_tile(by, dy, w.nty) * w.ntx + nb_tile(bx, dx, w.ntx);
  MC_GLOBAL int* now = glb(w.tl_cnt) + tile * kListCounts;
  MC_GLOBAL int* next = glb(w.tl_cnt_next) + tile * kListCounts;
  int at = tile * w.tl_stride + segment_first(w, seg), cap = segment_cap(w, seg);
  int n = own ? now[kCntOwn] + now[kCntStrays] : now[seg];
  if (own ? n > cap : (w.tl_kind == kSegments && nearly_full(n, cap))) {
    if (!own) n += (n >> 2) + 8;
    const int a = atomicAdd((int*)(list_words(w, glb(w.tl_cnt)) + kWordSpill), n);
    if (a >= 0 && n <= w.tl_spill - a) {         // (none left: nodes that do not fit flag the tiles they are for)
      at = w.ntx * w.nty * w.tl_stride + a;
      cap = n;
    }
  }
  next[kFirst + seg] = at;
  next[seg] = cap;
}

template <int TILE, int NT>
static __device__ __forceinline__ void filter_tile(const WorldDev& w, int packed, unsigned char* smem,
                                                   int window_bytes) {
  using C = TileCfg<TILE>;
  constexpr int kRing = TILE + 2, kThreads = NT;
  unsigned long long* s_win = (unsigned long long*)smem;
  float* s_regf = (float*)(smem + window_bytes);
  float* s_mid = (float*)smem;
  const int tid = threadIdx.x;
  {
    const int R = w.radius, mode = w.mode;
    const int nx = w.nx, ny = w.ny;
    const int x0 = tile_x(packed) * TILE;
    const int y0 = tile_y(packed) * TILE;
    const int reg = kRing + 2 * R;
    const float inv_reg = 1.0f / (float)reg;
    const int xo = x0 - R - 1, yo = y0 - R - 1;   // region origin (unwrapped)
    float* s_st = s_mid + reg * kRing;
    if (C::kBinned && mode == kBinned) {
      const int tix = tile_y(packed) * w.ntx + tile_x(packed);
      const int S = reg + 6;                      // window side; window origin (xo - 3, yo - 3)
      const int P = S + kWinPad;                  // row pitch
      TileRecords<NT, 3, NT == 256 && TILE == 32 ? 3 : 2> nodes(w, tix);
      zero_lds_u64(s_win, S * P);
      if (w.tl_kind != kNoLists && w.ctl_src->remaining > 1) {
        if (tid == 0) {                           // (the other numbers have one writer each)
          MC_GLOBAL int* next = glb(w.tl_cnt_next);
          next[tix * kListCounts + kCntStrays] = 0;
          next[tix * kListCounts + kCntFlags] = next[tix * kListCounts + kCntCrowded] = 0;
          if (tix == 0) list_words(w, next)[kWordSpill] = list_words(w, next)[kWordJump] = 0;
        }
        if (__builtin_expect(nodes.L.outgrows, 0)) reserve_segments(w, tile_x(packed), tile_y(packed));
      }
      const int ox = wrap_index(xo - 3, nx), oy = wrap_index(yo - 3, ny);
      const int keep_x = reg + 3 <= nx ? reg + 2 : nx;
      const int keep_y = reg + 3 <= ny ? reg + 2 : ny;
      __syncthreads();
      nodes.each(w, [&](const vi4& r, const vf2&) {
        const int dx = wrap_near((r.x & 0xffff) - 1 - ox, nx);
        const int dy = wrap_near((r.x >> 16) - 1 - oy, ny);
        if (dx > keep_x || dy > keep_y) return;
        unsigned qx[4], qy[4];
        peskin4_quant(__int_as_float(r.y), qx);
        peskin4_quant(__int_as_float(r.z), qy);
        unsigned long long* p = s_win + dy * P + dx;
#pragma unroll
        for (int b = 0; b < 4; ++b)
#pragma unroll
          for (int a = 0; a < 4; ++a) atomicAdd(p + b * P + a, weight_product(qx[a], qy[b]));
      });
      __syncthreads();
      const bool single = reg + 3 <= nx && reg + 3 <= ny;   // one image per needed cell
      for (int k = tid; k < reg * reg; k += kThreads) {
        const int r = div_small(k, inv_reg), c = k - r * reg;
        unsigned long long v;
        if (single) {
          v = s_win[(r + 3) * P + c + 3];
        } else {
          v = 0;
          for (int cy = first_image(r, ny); cy < S; cy += ny)
            for (int cx = first_image(c, nx); cx < S; cx += nx) v += s_win[cy * P + cx];
        }
        s_regf[k] = density_to_float(v);
      }
    } else if (mode == kSorted) {
      const MC_GLOBAL int* start = glb(w.start);
      const MC_GLOBAL vf4* rec = glbv<const vf4>(w.rec);
      for (int k = tid; k < reg * reg; k += kThreads) {
        const int r = div_small(k, inv_reg), c = k - r * reg;
        s_regf[k] = gather_density(start, rec, nx, ny, wrap_index(xo + c, nx), wrap_index(yo + r, ny));
      }
    } else {
      const MC_GLOBAL float* sd = glb(w.s);
      for (int k = tid; k < reg * reg; k += kThreads) {
        const int r = div_small(k, inv_reg), c = k - r * reg;
        s_regf[k] = sd[(size_t)wrap_index(yo + r, ny) * nx + wrap_index(xo + c, nx)];
      }
    }
    float g[kMaxRadius + 1];
#pragma unroll
    for (int m = 0; m <= kMaxRadius; ++m) g[m] = w.gtap[m];
    __syncthreads();
    switch (R) {                                  // uniform: the world's radius
      case 1: filter_passes<TILE, NT, 1>(s_regf, s_mid, s_st, g); break;
      case 2: filter_passes<TILE, NT, 2>(s_regf, s_mid, s_st, g); break;
      case 3: filter_passes<TILE, NT, 3>(s_regf, s_mid, s_st, g); break;
      case 4: filter_passes<TILE, NT, 4>(s_regf, s_mid, s_st, g); break;
      case 5: filter_passes<TILE, NT, 5>(s_regf, s_mid, s_st, g); break;
      case 6: filter_passes<TILE, NT, 6>(s_regf, s_mid, s_st, g); break;
      case 7: filter_passes<TILE, NT, 7>(s_regf, s_mid, s_st, g); break;
      default: filter_passes<TILE, NT, 8>(s_regf, s_mid, s_st, g); break;
    }
    MC_GLOBAL vf2* grad = glbv<vf2>(w.grad);
    for (int k = tid; k < TILE * TILE; k += kThreads) {
      const int r = k >> C::kShift, c = k & (TILE - 1);
      const int gx = x0 + c, gy = y0 + r;
      if (gx < nx && gy < ny) {
        const float* p = s_st + (r + 1) * kRing + (c + 1);
        const vf2 gr = {0.5f * (p[1] - p[-1]), 0.5f * (p[kRing] - p[-kRing])};
        grad[(size_t)gy * nx + gx] = gr;
      }
    }
  }
}

template <int TILE>
__global__ __launch_bounds__(TileCfg<TILE>::kThreads) void k_filter(const WorldDev* __restrict__ W, Tables T,
                                                                     int window_bytes) {
  extern __shared__ __align__(16) unsigned char smem[];
  const XcdLoop tiles(n_tiles<TILE>(T));
  for (int it = tiles.first; it < tiles.end; it += tiles.step) {
    const int2 tl = tile_entry<TILE>(T, it);
    const WorldDev& w = W[tl.x];
    if (w.ctl_src->remaining <= 0) continue;
    filter_tile<TILE, TileCfg<TILE>::kThreads>(w, tl.y, smem, window_bytes);
    __syncthreads();
  }
}

// S0 - S3 of binned worlds in one launch: the elastic force and the filter both
// follow from the step's positions alone, so pack blocks and tile blocks run
// side by side (a pack block waits at barriers and for its neighbours' data
// most of its time, a tile block issues).  Rounds of eight blocks, one per
// XCD, alternate between the two kinds until one has run out.
template <int TILE, int PACK, bool GEN, bool BR>
__global__ __launch_bounds__(PACK) void k_prepare(const WorldDev* __restrict__ W, Tables T, int window_bytes,
                                                  int tile_rounds, int pack_rounds) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int round = blockIdx.x >> 3, x = blockIdx.x & 7, both = 2 * min(tile_rounds, pack_rounds);
  const bool tile_role = round < both ? (round & 1) != 0 : tile_rounds > pack_rounds;
  const int b = ((round < both ? round >> 1 : round - (both >> 1)) << 3) + x;
  if (tile_role) {
    const XcdLoop tiles(n_tiles<TILE>(T), b, tile_rounds << 3);
    for (int it = tiles.first; it < tiles.end; it += tiles.step) {
      const int2 tl = tile_entry<TILE>(T, it);
      const WorldDev& w = W[tl.x];
      if (w.ctl_src->remaining <= 0) continue;
      filter_tile<TILE, PACK>(w, tl.y, smem, window_bytes);
      __syncthreads();
    }
  } else {
    const XcdLoop packs(*T.n_packs, b, pack_rounds << 3);
    for (int it = packs.first; it < packs.end; it += packs.step) {
      const Pack pk = T.packs[it];
      const WorldDev& w = W[pk.world];
      const Ctl ctl = *w.ctl_src;
      if (ctl.remaining <= 0) continue;
      elastic_pack<PACK, GEN, BR>(w, pk, ctl, *(ElasticLds<PACK, BR>*)smem);
      __syncthreads();
    }
  }
}

// ---------------------------------------------------------------------------
// S4: repulsion F_rep = -k_rep sum_c W(c - x) G_c and the total node force.
// Direct mode also spreads it with global atomics; sorted mode runs in slot
// order and stores the node records.
// ---------------------------------------------------------------------------
template <int PACK>
__global__ __launch_bounds__(PACK) void k_repulse(const WorldDev* __restrict__ W, Tables T) {
  const int npk = *T.n_packs;
  for (int it = blockIdx.x; it < npk; it += gridDim.x) {
    const Pack pk = T.packs[it];
    const WorldDev& w = W[pk.world];
    if (w.mode == kBinned || w.ctl_src->remaining <= 0) continue;   // binned: in k_spread
    const int sl = pk.node_begin + threadIdx.x;      // node index, or sorted slot
    if (sl >= pk.node_end) continue;
    const int mode = w.mode;
    const int gi = mode == kSorted ? glb(w.perm)[sl] : sl;
    const int N = w.n_part;
    const int nx = w.nx, ny = w.ny;
    const MC_GLOBAL int* cell = glb(w.cell_in);
    const MC_GLOBAL float* frac = glb(w.frac_in);
    const MC_GLOBAL vf2* grad = glbv<const vf2>(w.grad);
    MC_GLOBAL float* fel = glb(w.fel);
    const int bx = wrap_index(cell[gi], nx);
    const int by = wrap_index(cell[N + gi], ny);
    const float fx = frac[gi], fy = frac[N + gi];
    float wx[4], wy[4];
    peskin4(fx, wx);
    peskin4(fy, wy);
    int ix[4];
#pragma unroll
    for (int a = 0; a < 4; ++a) ix[a] = wrap_near(bx - 1 + a, nx);
    float gx = 0.f, gy = 0.f;
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const MC_GLOBAL vf2* row = grad + (size_t)wrap_near(by - 1 + b, ny) * nx;
      float rx = 0.f, ry = 0.f;
#pragma unroll
      for (int a = 0; a < 4; ++a) {
        const vf2 g = row[ix[a]];
        rx += wx[a] * g.x;
        ry += wx[a] * g.y;
      }
      gx += wy[b] * rx;
      gy += wy[b] * ry;
    }
    const MC_GLOBAL float* fe = glb(w.fel_el);
    const float Fx = fe[gi] - w.k_rep * gx;
    const float Fy = fe[N + gi] - w.k_rep * gy;
    fel[gi] = Fx;
    fel[N + gi] = Fy;
    if (mode == kSorted) {
      const vf4 r = {fx, fy, Fx, Fy};
      glbv<vf4>(w.rec)[sl] = r;
    } else if (mode == kDirect && w.d_marker) {
      // two layers: half of the force from each marker
      const float dx = glb(w.d_marker)[gi], dy = glb(w.d_marker)[N + gi];
      const int cx = cell[gi], cy = cell[N + gi];
#pragma unroll
      for (int sgn = 1; sgn >= -1; sgn -= 2) {
        int hx, hy;
        float mx, my;
        marker_home(cx, fx, sgn * dx, nx, &hx, &mx);
        marker_home(cy, fy, sgn * dy, ny, &hy, &my);
        atomic_spread_vec(glb((float*)w.Fg), nx, ny, hx, hy, mx, my, 0.5f * Fx, 0.5f * Fy);
      }
    } else if (mode == kDirect) {
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        MC_GLOBAL float* row = glb((float*)w.Fg) + 2 * (size_t)wrap_near(by - 1 + b, ny) * nx;
#pragma unroll
        for (int a = 0; a < 4; ++a) {
          const float ww = wx[a] * wy[b];
          unsafeAtomicAdd((float*)(row + 2 * ix[a]), ww * Fx);
          unsafeAtomicAdd((float*)(row + 2 * ix[a] + 1), ww * Fy);
        }
      }
    }
  }
}

// Fluid velocity of a cell from its shifted populations g (the lattice weights
// have zero first moment, so the shift does not change the momentum sum) and
// its grid force F; drho = rho - 1.
static __device__ __forceinline__ vf2 fluid_velocity(const float* g, const vf2& F, float* drho) {
  const float d = ((g[0] + g[1]) + (g[2] + g[3])) + ((g[4] + g[5]) + (g[6] + g[7])) + g[8];
  const float jx = (g[1] - g[3]) + (g[5] - g[6]) + (g[8] - g[7]);
  const float jy = (g[2] - g[4]) + (g[5] - g[8]) + (g[6] - g[7]);
  const float inv = 1.0f / (1.0f + d);
  *drho = d;
  const vf2 u = {(jx + 0.5f * F.x) * inv, (jy + 0.5f * F.y) * inv};
  return u;
}

// Pushes the post-collision populations of cell (x, y) to its neighbours.  The
// wrapped rows and columns are formed once (in the loop over q the compiler
// formed them per population: 247 vector instructions a
// wavefront of k_lbm, now 221).
template <class Store>
static __device__ __forceinline__ void push(int x, int y, int nx, int ny, const float* out, Store store) {
  const int xs[3] = {x > 0 ? x - 1 : nx - 1, x, x + 1 < nx ? x + 1 : 0};
  const int rows[3] = {(y > 0 ? y - 1 : ny - 1) * nx, y * nx, (y + 1 < ny ? y + 1 : 0) * nx};
  static_for<9>([&](auto qq) {
    constexpr int q = qq, cx = (q == 1 || q == 5 || q == 8) - (q == 3 || q == 6 || q == 7),
                  cy = (q == 2 || q == 5 || q == 6) - (q == 4 || q == 7 || q == 8);
    store(q, rows[cy + 1] + xs[cx + 1], out[q]);
  });
}

// Post-collision populations of a cell.  Equilibrium minus weights: w_q (drho +
// rho (3 cu + 4.5 cu^2 - 1.5 u^2)); Guo source: w_q (3 (c - u) + 9 (c.u) c) . F;
// split into the parts symmetric and antisymmetric under q <-> opposite(q).
static __device__ __forceinline__ void collide(const WorldDev& w, const float* g, const vf2& F, const vf2& u,
                                               float drho, float* out) {
  const float Fx = F.x, Fy = F.y, ux = u.x, uy = u.y;
  const float rho = 1.0f + drho;
  const float usq = ux * ux + uy * uy;
  const float op = w.om_p, om = w.om_m;
  const float sp = 1.0f - 0.5f * op, sm = 1.0f - 0.5f * om;
  const float base = 1.5f * usq;
  const float uF = ux * Fx + uy * Fy;
  {
    const float w0 = 4.0f / 9.0f;
    const float geq0 = w0 * (drho - rho * base);
    const float S0 = w0 * (-3.0f * uF);
    out[0] = g[0] - op * (g[0] - geq0) + sp * S0;
  }
#pragma unroll
  for (int pr = 0; pr < 4; ++pr) {
    const int q = pr < 2 ? 1 + pr : 5 + (pr - 2);
    const int qb = q + 2;
    const float wq = pr < 2 ? (1.0f / 9.0f) : (1.0f / 36.0f);
    const float cxq = (float)kCX[q], cyq = (float)kCY[q];
    const float cu = cxq * ux + cyq * uy;
    const float cF = cxq * Fx + cyq * Fy;
    const float eqp = wq * (drho + rho * (4.5f * cu * cu - base));
    const float eqm = wq * rho * 3.0f * cu;
    const float Sp = wq * (9.0f * cu * cF - 3.0f * uF);
    const float Sm = wq * 3.0f * cF;
    const float gp = 0.5f * (g[q] + g[qb]);
    const float gm = 0.5f * (g[q] - g[qb]);
    const float relp = -op * (gp - eqp) + sp * Sp;
    const float relm = -om * (gm - eqm) + sm * Sm;
    out[q] = g[q] + relp + relm;
    out[qb] = g[qb] + relp - relm;
  }
}

// ---------------------------------------------------------------------------
// S5: grid force of a tile, summed in LDS over the tile's list (binned)
// or by fixed-order gathers over sorted segments (sorted); every cell of the
// tile is written once.  Direct mode accumulates in k_repulse instead.
// ---------------------------------------------------------------------------
// MK: the two-layer variant (binned worlds with markers, which the plain
// variant skips): the gradient is staged one cell wider on every side and
// the nodes spread through their markers.
template <int TILE, bool MK>
__global__ __launch_bounds__(TileCfg<TILE>::kThreads) void k_spread(const WorldDev* __restrict__ W, Tables T) {
  using C = TileCfg<TILE>;
  using SW = SpreadWin<TILE>;
  constexpr int kThreads = C::kThreads;
  constexpr int kGSide = MK ? SW::kGSide : SW::kSide, kGCells = kGSide * kGSide;
  __shared__ __align__(16) long long s_fx[SW::kCells];   // 64-bit fixed point, padded window
  __shared__ __align__(16) long long s_fy[SW::kCells];
  __shared__ vf2 s_g[kGCells];                  // gradient over the window (binned)
  const int nt = n_tiles<TILE>(T);
  const int tid = threadIdx.x;
  const XcdLoop tiles(nt);
  for (int it = tiles.first; it < tiles.end; it += tiles.step) {
    const int2 tl = tile_entry<TILE>(T, it);
    const WorldDev& w = W[tl.x];
    if (w.mode == kDirect || w.ctl_src->remaining <= 0) continue;
    if (MK != (w.mode == kBinned && w.d_marker != nullptr)) continue;
    const int mode = w.mode;
    const int nx = w.nx, ny = w.ny;
    const int x0 = tile_x(tl.y) * TILE;
    const int y0 = tile_y(tl.y) * TILE;
    const int tw = min(TILE, nx - x0), th = min(TILE, ny - y0);
    if (C::kBinned && mode == kBinned) {
      const int tix = tile_y(tl.y) * w.ntx + tile_x(tl.y);
      // S4 repulsion is formed here, per node, from the gradient staged over
      // the window (grid cells (x0 - 3 + i, y0 - 3 + j), periodic)
      // (the gradient's loads first: they need no other, and loads return in order)
      const WindowLoads<kThreads, kGSide> grad(glbv<const vf2>(w.grad), nx, ny, x0 - (MK ? 4 : 3), y0 - (MK ? 4 : 3));
      SpreadNodes<TILE> nodes(w, tix, glb(w.fel_el));
      zero_lds_u64(s_fx, SW::kCells);
      zero_lds_u64(s_fy, SW::kCells);
      grad.store(s_g);
      __syncthreads();
      if constexpr (MK)
        tile_spread_markers<TILE, true>(w, nodes, x0, y0, tw, th, 1.0f, s_fx, s_fy, s_g);
      else
        tile_spread_vec<TILE, true>(w, nodes, x0, y0, tw, th, 1.0f, s_fx, s_fy, s_g);
      __syncthreads();
    }
    MC_GLOBAL vf2* Fg = glbv<vf2>(w.Fg);
    const MC_GLOBAL int* start = glb(w.start);
    const MC_GLOBAL vf4* rec = glbv<const vf4>(w.rec);
    for (int k = tid; k < TILE * TILE; k += kThreads) {
      const int ly = k >> C::kShift, lx = k & (TILE - 1);
      if (lx >= tw || ly >= th) continue;
      vf2 F;
      if (C::kBinned && mode == kBinned) {
        F.x = fix_to_float(spread_cell<SW::kSide>(s_fx, lx, ly, nx, ny));
        F.y = fix_to_float(spread_cell<SW::kSide>(s_fy, lx, ly, nx, ny));
      } else {
        F = gather_force(start, rec, nx, ny, x0 + lx, y0 + ly);
      }
      Fg[(size_t)(y0 + ly) * nx + x0 + lx] = F;
    }
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------
// S6: D2Q9 two-relaxation-time collision with Guo forcing and push streaming
// over 256 contiguous cells per item.  Populations are stored shifted
// (g = f - w_q) so FP32 resolves the small deviations from rest.  Writes u;
// sets the world flag on NaN or |u| > u_max.  In direct mode it also clears
// the HBM accumulators for the next step.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_lbm(const WorldDev* __restrict__ W, Tables T) {
  constexpr int CPT = kCellsPerItem / 256;      // cells per thread, loaded together
  const XcdLoop items(*T.n_items);
  for (int it = items.first; it < items.end; it += items.step) {
    const int2 item = T.items[it];
    const WorldDev& w = W[item.x];
    const Ctl cs = *w.ctl_src;
    const bool live = cs.remaining > 0;
    if (item.y == 0 && threadIdx.x == 0) {
      Ctl cd = cs;
      if (live) { cd.t += 1; cd.remaining -= 1; }
      *w.ctl_dst = cd;
    }
    if (!live) continue;
    const int nx = w.nx, ny = w.ny;
    const int ncell = nx * ny;
    const int ry = item.y / nx;                 // row and column of the item's first cell
    const int rx = item.y - ry * nx;
    const MC_GLOBAL float* src = glb(w.f_src);
    MC_GLOBAL float* dst = glb(w.f_dst);
    float gg[CPT][9];
    vf2 FF[CPT];
#pragma unroll
    for (int h = 0; h < CPT; ++h) {             // every load of every cell first
      const int c = min(item.y + (int)threadIdx.x + 256 * h, ncell - 1);
#pragma unroll
      for (int q = 0; q < 9; ++q)                 // read once per step: no cache allocation
        gg[h][q] = __builtin_nontemporal_load((const float*)(src + (size_t)q * ncell + c));
      FF[h] = glbv<vf2>(w.Fg)[c];
    }
#pragma unroll
    for (int h = 0; h < CPT; ++h) {
      const int c = item.y + (int)threadIdx.x + 256 * h;
      if (c >= ncell) continue;
      int x = rx + (int)threadIdx.x + 256 * h, y = ry;
      while (x >= nx) {                           // items may run over row ends
        x -= nx;
        ++y;
      }
      const float* g = gg[h];
      const vf2 F = FF[h];
      if (w.mode == kDirect) {
        const vf2 zero = {0.f, 0.f};
        glbv<vf2>(w.Fg)[c] = zero;
        glb(w.s)[c] = 0.f;
      }
      float drho, out[9];
      const vf2 uv = fluid_velocity(g, F, &drho);
      glbv<vf2>(w.u)[c] = uv;
      if (!(uv.x * uv.x + uv.y * uv.y <= w.u_max2)) atomicOr((unsigned*)glb(w.flags), kFlagUnstable);
      collide(w, g, F, uv, drho, out);
      // (non-temporal: the next read is a step away; the caches keep what the
      // following kernels read instead)
      push(x, y, nx, ny, out, [&](int q, int c, float v) {
        __builtin_nontemporal_store(v, (float*)(dst + (size_t)q * ncell) + c);
      });
    }
  }
}



// ---------------------------------------------------------------------------
// S7: gather the step's fluid velocity at each node and integrate
// (x <- x + sum_c W(c - x) u(c)), carrying the fraction into the cell.
// ---------------------------------------------------------------------------
template <int PACK>
__global__ __launch_bounds__(PACK) void k_integrate(const WorldDev* __restrict__ W, Tables T) {
  const int npk = *T.n_packs;
  for (int it = blockIdx.x; it < npk; it += gridDim.x) {
    const Pack pk = T.packs[it];
    const WorldDev& w = W[pk.world];
    if (w.mode == kBinned || w.ctl_src->remaining <= 0) continue;   // binned: k_integrate_tile
    const int gi = pk.node_begin + threadIdx.x;
    if (gi >= pk.node_end) continue;
    const int N = w.n_part;
    const int nx = w.nx, ny = w.ny;
    const MC_GLOBAL int* cell = glb(w.cell_in);
    const MC_GLOBAL float* frac = glb(w.frac_in);
    const MC_GLOBAL vf2* u = glbv<const vf2>(w.u);
    const int cx = cell[gi], cy = cell[N + gi];
    const float fx = frac[gi], fy = frac[N + gi];
    const int bx = wrap_index(cx, nx), by = wrap_index(cy, ny);
    float wx[4], wy[4];
    peskin4(fx, wx);
    peskin4(fy, wy);
    int ix[4];
#pragma unroll
    for (int a = 0; a < 4; ++a) ix[a] = wrap_near(bx - 1 + a, nx);
    float dux = 0.f, duy = 0.f;
    if (w.d_marker) {
      // two layers: the mean of the markers' interpolated velocities
      const float dx = glb(w.d_marker)[gi], dy = glb(w.d_marker)[N + gi];
#pragma unroll
      for (int sgn = 1; sgn >= -1; sgn -= 2) {
        int hx, hy;
        float mx, my;
        marker_home(cx, fx, sgn * dx, nx, &hx, &mx);
        marker_home(cy, fy, sgn * dy, ny, &hy, &my);
        const vf2 v = gather_vec(u, nx, ny, hx, hy, mx, my);
        dux += 0.5f * v.x;
        duy += 0.5f * v.y;
      }
    } else {
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const MC_GLOBAL vf2* row = u + (size_t)wrap_near(by - 1 + b, ny) * nx;
      float ax = 0.f, ay = 0.f;
#pragma unroll
      for (int a = 0; a < 4; ++a) {
        const vf2 v = row[ix[a]];
        ax += wx[a] * v.x;
        ay += wx[a] * v.y;
      }
      dux += wy[b] * ax;
      duy += wy[b] * ay;
    }
    }
    float nfx = fx + dux, nfy = fy + duy;
    const float flx = floorf(nfx), fly = floorf(nfy);
    int ncx = cx + (int)flx, ncy = cy + (int)fly;
    nfx -= flx;
    nfy -= fly;
    if (nfx >= 1.0f) { nfx = 0.0f; ncx += 1; }
    if (nfy >= 1.0f) { nfy = 0.0f; ncy += 1; }
    MC_GLOBAL int* cell_out = glb(w.cell_out);
    MC_GLOBAL float* frac_out = glb(w.frac_out);
    cell_out[gi] = ncx;
    cell_out[N + gi] = ncy;
    frac_out[gi] = nfx;
    frac_out[N + gi] = nfy;
  }
}

// ---------------------------------------------------------------------------
// Binned worlds: the node gather of S7 (u) per tile.  The field is staged in
// LDS for the tile plus the support margin (cells x0-1 .. x0+TILE+1)
// with coalesced loads; every node whose home cell lies in the tile (its own)
// gathers its 4x4 window from LDS.  (The S4 gather of binned worlds happens
// inside k_spread.)
// ---------------------------------------------------------------------------
// The field is staged over the cells (x0 - 1 - E .. x0 + TILE + 1 + E) of each
// axis (side TILE + 3 + 2E): every support of a node whose home lies in the
// tile (E = 0), or of its two-layer markers (E = 1: a marker's home lies
// within one cell of its node's).
// 4x4 kernel-weighted sum of a staged vector field
// at a point whose support starts at staged cell (lx, ly) (a node with home
// cell (lx, ly) of the tile when E = 0; weights wx, wy along x and y).
template <int TILE, int E = 0>
__device__ __forceinline__ vf2 gather_staged(const vf2* st, int lx, int ly, const float* wx, const float* wy) {
  constexpr int kStage = TILE + 3 + 2 * E;
  float gx = 0.f, gy = 0.f;
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    const vf2* row = st + (ly + b) * kStage + lx;
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
  const vf2 out = {gx, gy};
  return out;
}

// Next step's lists from the block that integrated tile (bx, by): cursors of
// the tile's own segment and of its segments in the eight neighbours' lists
// (at kCntNear and kCntFar + q: in the list of the tile it is neighbour q of).
template <int TILE>
struct AppendLds {
  static constexpr int kAxis = TILE + 2 * kSmallMove;
  int cur[kSegs];
  int2 place[kSegs];                             // where each segment begins, and how many it takes
  unsigned char axis[2 * kAxis];                 // axis_pairs of the places along x, then y
};
template <int TILE>
static __device__ __forceinline__ void init_append(const WorldDev& w, int bx, int by, AppendLds<TILE>& lds) {
  constexpr int kAxis = AppendLds<TILE>::kAxis;
  const int seg = threadIdx.x;
  if (seg < 2 * kAxis) {
    const bool y = seg >= kAxis;
    const int l = seg - (y ? kAxis : 0) - kSmallMove;
    lds.axis[seg] = (unsigned char)axis_pairs(axis_classes(Reach(w), l, y ? min(TILE, w.ny - by * TILE) : min(TILE, w.nx - bx * TILE),
                                            y ? w.nty : w.ntx));
  }
  if (seg >= kSegs) return;
  const bool own = seg < kCntNear;
  const int q = (seg - kCntNear) & 7, dx = own ? 0 : nb_dx(q), dy = own ? 0 : nb_dy(q);
  const int tile = nb_tile(by, dy, w.nty) * w.ntx + nb_tile(bx, dx, w.ntx);
  lds.cur[seg] = 0;
  lds.place[seg] = make_int2(tile * w.tl_stride + segment_first(w, seg), segment_cap(w, seg));
}
// The places that the filter left in the next lists (reserve_segments).  By every
// thread after its own init_append, before the barrier ahead of append_nodes.
template <int TILE>
static __device__ __forceinline__ void take_places(const WorldDev& w, int bx, int by, AppendLds<TILE>& lds) {
  const int seg = threadIdx.x;
  if (seg >= kSegs) return;
  const int q = (seg - kCntNear) & 7, dx = seg < kCntNear ? 0 : nb_dx(q), dy = seg < kCntNear ? 0 : nb_dy(q);
  if (seg == kCntStrays || !nb_exists(dx, w.ntx) || !nb_exists(dy, w.nty)) return;
  const MC_GLOBAL int* c = glb(w.tl_cnt_next) + (nb_tile(by, dy, w.nty) * w.ntx + nb_tile(bx, dx, w.ntx)) * kListCounts;
  lds.place[seg] = make_int2(c[kFirst + seg], c[seg]);
}
// Record `slot` of the segment, or the flags of the lists that cannot be used
// without it.
static __device__ __forceinline__ void append_record(const WorldDev& w, MC_GLOBAL vi4* lists, MC_GLOBAL int* counts,
                                                     int2 place, int tx, int ty, int seg, int slot, const vi4& rec) {
  if (__builtin_expect(slot < place.y, 1)) lists[place.x + slot] = rec;
  else flag_overflow(w, counts, tx, ty, seg);
}

// Appends up to PER nodes per thread (node index -1: none) to the lists of the
// tiles they reach; called by every lane.
template <int TILE, int PER>
static __device__ __forceinline__ void append_nodes(const WorldDev& w, int bx, int by, const vi4* rec,
                                                    AppendLds<TILE>& lds) {
  constexpr int kAxis = AppendLds<TILE>::kAxis;
  const int ntx = w.ntx, nty = w.nty;
  MC_GLOBAL vi4* lists = glbv<vi4>(w.tl_rec_next);
  MC_GLOBAL int* counts = glb(w.tl_cnt_next);
  const auto jump = [&](const Place& pl) {
    if (pl.lx < -kSmallMove || pl.lx >= min(TILE, w.nx - bx * TILE) + kSmallMove || pl.ly < -kSmallMove ||
        pl.ly >= min(TILE, w.ny - by * TILE) + kSmallMove)
      atomicOr((int*)(list_words(w, counts) + kWordJump), 1);
  };
#pragma unroll
  for (int p = 0; p < PER; ++p) {
    const vi4& r = rec[p];
    const bool has = r.w >= 0;
    const unsigned long long m = __ballot(has);
    if (!m) continue;
    // own segment: one LDS atomic per wavefront
    const int lane = __lane_id(), leader = __ffsll(m) - 1;
    int k = 0;
    if (lane == leader) k = atomicAdd(&lds.cur[kCntOwn], __popcll(m));
    const int2 place = lds.place[kCntOwn];
    const Place pl(w, TILE, bx, by, r.x & 0xffff, r.x >> 16);
    const int ix = pl.inside ? pl.lx + kSmallMove : 0, iy = kAxis + (pl.inside ? pl.ly + kSmallMove : 0);
    const Pairs a(lds.axis[ix], lds.axis[iy], !pl.inside);
    k = __shfl(k, leader) + __popcll(m & ((1ull << lane) - 1ull));
    if (!has) continue;
    if (__builtin_expect(w.tl_kind != kSegments, 0)) {   // own nodes alone
      if (k < place.y) write_entry(w, lists, place.x + k, r);
      else flag_overflow(w, counts, bx, by, kCntOwn);
      const int tx = (r.x & 0xffff) >> TileCfg<TILE>::kShift, ty = (r.x >> 16) >> TileCfg<TILE>::kShift;
      if (tx != bx || ty != by) {                // (counted, so that its block knows how many it gets)
        atomicAdd((int*)(counts + (ty * ntx + tx) * kListCounts + kCntStrays), 1);
        jump(pl);
      }
      continue;
    }
    if (__builtin_expect(!__any(a.more), 1)) {
      // every lane for its own neighbours at once, slots and places fetched together
      // (512^2, 65,536 nodes: 28.8 -> 28.5 us per step)
      const int q1 = class_segment(a.side_x, a.qx()), q2 = class_segment(a.side_y, a.qy()),
                q3 = class_segment(a.corner, a.qc());
      const auto listed = [](int cls) { return cls == 1 || cls == 2; };
      int k1 = 0, k2 = 0, k3 = 0;
      int2 p1, p2, p3;
      if (listed(a.side_x)) k1 = atomicAdd(&lds.cur[q1], 1), p1 = lds.place[q1];
      if (listed(a.side_y)) k2 = atomicAdd(&lds.cur[q2], 1), p2 = lds.place[q2];
      if (listed(a.corner)) k3 = atomicAdd(&lds.cur[q3], 1), p3 = lds.place[q3];
      append_record(w, lists, counts, place, bx, by, kCntOwn, k, r);
      const int tx = nb_tile(bx, a.dx, ntx), ty = nb_tile(by, a.dy, nty);
      if (listed(a.side_x)) append_record(w, lists, counts, p1, tx, by, q1, k1, r);
      if (listed(a.side_y)) append_record(w, lists, counts, p2, bx, ty, q2, k2, r);
      if (listed(a.corner)) append_record(w, lists, counts, p3, tx, ty, q3, k3, r);
      if (__builtin_expect(a.side_x == 0 || a.side_y == 0 || a.corner == 0, 0))   // it has left for that one
        append_stray(w, lists, counts, a.side_y == 0 ? bx : tx, a.side_x == 0 ? by : ty, r);
      continue;
    }
    append_record(w, lists, counts, place, bx, by, kCntOwn, k, r);
    const Classes c = neighbour_classes<TILE>(w, bx, by, r.x & 0xffff, r.x >> 16);
#pragma unroll 1
    for (int q = 0; q < 8; ++q) {
      const int cls = c.of(q), tx = nb_tile(bx, nb_dx(q), ntx), ty = nb_tile(by, nb_dy(q), nty);
      if (cls > 2) continue;
      if (cls == 0) {
        append_stray(w, lists, counts, tx, ty, r);
        continue;
      }
      const int seg = class_segment(cls, q);
      append_record(w, lists, counts, lds.place[seg], tx, ty, seg, atomicAdd(&lds.cur[seg], 1), r);
    }
    if (c.beyond) {
      jump(pl);
      append_strays<TILE>(w, lists, counts, bx, by, r);
    }
  }
}

// The numbers and places of the segments this block wrote (after a barrier).
template <int TILE>
static __device__ __forceinline__ void store_counts(const WorldDev& w, int bx, int by, const AppendLds<TILE>& lds) {
  const int seg = threadIdx.x;
  if (seg == kCntStrays || seg >= kSegs) return;
  const int q = (seg - kCntNear) & 7;
  const int dx = seg < kCntNear ? 0 : nb_dx(q), dy = seg < kCntNear ? 0 : nb_dy(q);
  if (!nb_exists(dx, w.ntx) || !nb_exists(dy, w.nty)) return;
  MC_GLOBAL int* c = glb(w.tl_cnt_next) + (nb_tile(by, dy, w.nty) * w.ntx + nb_tile(bx, dx, w.ntx)) * kListCounts;
  const int n = lds.cur[seg], at = lds.place[seg].x;
  c[seg] = n;
  c[kFirst + seg] = at;
  // (in the spill area: the next step's may have to be there as well)
  if (__builtin_expect(nearly_full(n, lds.place[seg].y) || at >= w.ntx * w.nty * w.tl_stride, 0))
    glb(w.tl_cnt_next)[(by * w.ntx + bx) * kListCounts + kCntCrowded] = 1;
}

// A tile's nodes for its integration (its own and the strays): records and
// unwrapped cells of up to kOwnPer nodes per thread, loaded together (the
// first round's beside the staging of the velocity).  Every wavefront goes
// through its share of them on its own.
constexpr int kOwnPer = 2;
template <int TILE>
struct OwnNodes {
  static constexpr int NT = TileCfg<TILE>::kThreads;
  WaveRuns<NT, 1> L;
  vi4 r[kOwnPer];
  int cx[kOwnPer], cy[kOwnPer];
  __device__ __forceinline__ void load(const WorldDev& w, int base) {
    int e[kOwnPer];
#pragma unroll
    for (int q = 0; q < kOwnPer; ++q)              // clamped, so that every load is issued at once
      e[q] = L.d0 + min(base + q * 64 + (int)(threadIdx.x & 63), L.total - 1);
    if (__builtin_expect(!unlisted(w), 1)) {
#pragma unroll
      for (int q = 0; q < kOwnPer; ++q) r[q] = glbv<const vi4>(w.tl_rec)[e[q]];
#pragma unroll
      for (int q = 0; q < kOwnPer; ++q) {
        cx[q] = glb(w.cell_in)[r[q].w];
        cy[q] = glb(w.cell_in)[w.n_part + r[q].w];
      }
      return;
    }
#pragma unroll
    for (int q = 0; q < kOwnPer; ++q) {
      const int gi = L.mode == kModeAll ? e[q] : glb((const int*)w.tl_rec)[e[q]];
      cx[q] = glb(w.cell_in)[gi];
      cy[q] = glb(w.cell_in)[w.n_part + gi];
      r[q].y = __float_as_int(glb(w.frac_in)[gi]);
      r[q].z = __float_as_int(glb(w.frac_in)[w.n_part + gi]);
      r[q].w = gi;
    }
  }
  // Whether the entries are nodes alone.
  __device__ __forceinline__ bool unlisted(const WorldDev& w) const {
    return L.mode == kModeAll || (L.mode == kModeAround && w.tl_kind == kOwnIndices);
  }
  __device__ __forceinline__ OwnNodes(const WorldDev& w, int tile) : L(wave_runs<NT, 1>(w, tile)) {
    if (L.total > 0) load(w, 0);
  }
};

// S7 of a tile's own nodes (o: the first round's, loaded), from the velocity
// staged in s_u: the new positions and, unless this is the run's last step
// (append), the next step's lists.  The cursors have been cleared.
template <int TILE, bool MK>
static __device__ __forceinline__ void integrate_own(const WorldDev& w, OwnNodes<TILE>& o, int packed, bool append,
                                                     const vf2* s_u, AppendLds<TILE>& lds) {
  const int nx = w.nx, ny = w.ny, N = w.n_part;
  const int x0 = tile_x(packed) * TILE, y0 = tile_y(packed) * TILE;
  const int tw = min(TILE, nx - x0), th = min(TILE, ny - y0);
  const int tile = tile_y(packed) * w.ntx + tile_x(packed);
  bool loaded = true;                            // (the first round)
  do {
  for (int base = 0; base < o.L.total; base += kOwnPer * 64) {
    if (!loaded) o.load(w, base);
    loaded = false;
#pragma unroll
    for (int q = 0; q < kOwnPer; ++q) {
      vi4& r = o.r[q];
      const int home = wrap_index(o.cx[q], nx) | (wrap_index(o.cy[q], ny) << 16);
      bool has = base + q * 64 + (int)(threadIdx.x & 63) < o.L.total;
      if (o.unlisted(w)) r.x = home;
      if (has && r.x != home) atomicOr((unsigned*)glb(w.flags), kFlagLists);   // moved since its list was made
      const int lx = (r.x & 0xffff) - x0, ly = (r.x >> 16) - y0;   // (some only reach the tile, or left it)
      has = has && lx >= 0 && lx < tw && ly >= 0 && ly < th;
      if (!has) {
        r.w = -1;
        continue;
      }
      const float fx = __int_as_float(r.y), fy = __int_as_float(r.z);
      const int gi = r.w;
      float dux, duy;
      if constexpr (MK) {
        dux = duy = 0.f;
        const float ddx = glb(w.d_marker)[gi], ddy = glb(w.d_marker)[N + gi];
#pragma unroll
        for (int l = 0; l < 2; ++l) {
          const float sg = l == 0 ? 1.f : -1.f;
          int sx, sy;
          float mx, my;
          marker_shift(fx, sg * ddx, &sx, &mx);
          marker_shift(fy, sg * ddy, &sy, &my);
          float wx[4], wy[4];
          peskin4(mx, wx);
          peskin4(my, wy);
          const vf2 g = gather_staged<TILE, 1>(s_u, lx + sx + 1, ly + sy + 1, wx, wy);
          dux += g.x;
          duy += g.y;
        }
        dux *= 0.5f;
        duy *= 0.5f;
      } else {
        float wx[4], wy[4];
        peskin4(fx, wx);
        peskin4(fy, wy);
        const vf2 du = gather_staged<TILE>(s_u, lx, ly, wx, wy);
        dux = du.x;
        duy = du.y;
      }
      float nfx = fx + dux, nfy = fy + duy;
      const float flx = floorf(nfx), fly = floorf(nfy);
      int ncx = o.cx[q] + (int)flx, ncy = o.cy[q] + (int)fly;
      nfx -= flx;
      nfy -= fly;
      if (nfx >= 1.0f) { nfx = 0.0f; ncx += 1; }
      if (nfy >= 1.0f) { nfy = 0.0f; ncy += 1; }
      glb(w.cell_out)[gi] = ncx;
      glb(w.cell_out)[N + gi] = ncy;
      glb(w.frac_out)[gi] = nfx;
      glb(w.frac_out)[N + gi] = nfy;
      r.x = wrap_index(ncx, nx) | (wrap_index(ncy, ny) << 16);
      r.y = __float_as_int(nfx);
      r.z = __float_as_int(nfy);
    }
    if (append) append_nodes<TILE, kOwnPer>(w, tile_x(packed), tile_y(packed), o.r, lds);
  }
  } while (o.L.mode == kModeAround && o.L.next_run(w, tile));
  if (append) {
    __syncthreads();
    store_counts(w, tile_x(packed), tile_y(packed), lds);
  }
}

// MK: the two-layer variant (worlds with markers, which the plain variant
// skips): a node moves with the mean of its two markers' velocities.
template <int TILE, bool MK>
__global__ __launch_bounds__(TileCfg<TILE>::kThreads, MK && TILE == 32 ? 5 : 1) void k_integrate_tile(const WorldDev* __restrict__ W, Tables T) {
  constexpr int kE = MK ? 1 : 0;
  constexpr int kStage = TILE + 3 + 2 * kE, kThreads = TileCfg<TILE>::kThreads;
  __shared__ vf2 s_u[kStage * kStage];        // staged velocity, x and y interleaved
  __shared__ AppendLds<TILE> s_app;
  const int nt = n_tiles<TILE>(T);
  const XcdLoop tiles(nt);
  for (int it = tiles.first; it < tiles.end; it += tiles.step) {
    const int2 tl = tile_entry<TILE>(T, it);
    const WorldDev& w = W[tl.x];
    const int remaining = w.ctl_src->remaining;
    if (w.mode != kBinned || remaining <= 0) continue;
    if (MK != (w.d_marker != nullptr)) continue;
    const int nx = w.nx, ny = w.ny;
    const int x0 = tile_x(tl.y) * TILE;
    const int y0 = tile_y(tl.y) * TILE;
    const int tile = tile_y(tl.y) * w.ntx + tile_x(tl.y);
    const bool append = w.tl_kind != kNoLists && remaining > 1;
    if (append) init_append(w, tile_x(tl.y), tile_y(tl.y), s_app);
    const WindowLoads<kThreads, kStage> u(glbv<const vf2>(w.u), nx, ny, x0 - 1 - kE, y0 - 1 - kE);
    OwnNodes<TILE> own(w, tile);
    u.store(s_u);
    if (__builtin_expect(append && own.L.outgrows, 0)) take_places(w, tile_x(tl.y), tile_y(tl.y), s_app);
    __syncthreads();
    integrate_own<TILE, MK>(w, own, tl.y, append, s_u, s_app);
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------
// S4 - S7 of binned worlds without MDF in one tile kernel: the force spread
// over the tile and the cells its nodes' supports reach, the fluid update of
// the tile (and the velocity alone of the cells around it), and the
// integration of its nodes, with the grid force and the velocity in LDS
// throughout.  Where a launch lasts as long as its chain of dependent loads
// whatever its work, three chains and two launches less cost (TILE + 3)^2 /
// TILE^2 of the spread and of the population loads; where the populations stay
// in the caches the grid force (read and written), the velocity and the
// latencies saved count for more than that too.  Per step, separate kernels
// and this one: 1000 nodes on 128^2 (16-cell tiles) 25.3 and 17.5 us, 65,536 on
// 512^2 (16) 34.1 and 28.0, 262,144 on 1024^2 (32) 76.2 and 57.2.  Bound by
// the vector instructions it issues at the latter size.  16-cell tiles load
// their populations ahead of the spread (two cells a thread); 32-cell ones
// have five a thread, and with those in registers half as many wavefronts fit
// (1024^2: 75 us).  Non-temporal stores, which do k_lbm good, leave lines
// that two tiles share half written (1024^2: 71 us).
// The arithmetic is that of the separate kernels.
// ---------------------------------------------------------------------------
template <int TILE, bool MK>
__global__ __launch_bounds__(TileCfg<TILE>::kThreads, MK ? 3 : 4) void k_fluid_tile(const WorldDev* __restrict__ W, Tables T, int keep) {
  constexpr int kE = MK ? 1 : 0, LO = 1 + kE, HI = 2 + kE;
  using SW = SpreadWin<TILE, LO, HI>;
  constexpr int kThreads = TileCfg<TILE>::kThreads;
  constexpr int kStage = TILE + LO + HI, kCells = kStage * kStage, kIt = (kCells + kThreads - 1) / kThreads;
  constexpr int kGSide = MK ? SW::kGSide : SW::kSide;
  constexpr bool kAhead = TILE == 16;
  __shared__ __align__(16) long long s_fx[SW::kCells];
  __shared__ __align__(16) long long s_fy[SW::kCells];
  __shared__ vf2 s_g[kGSide * kGSide];          // density gradient, then the velocity
  __shared__ AppendLds<TILE> s_app;
  static_assert(kStage <= kGSide, "velocity in the gradient's place");
  const XcdLoop tiles(n_tiles<TILE>(T));
  for (int it = tiles.first; it < tiles.end; it += tiles.step) {
    const int2 tl = tile_entry<TILE>(T, it);
    const WorldDev& w = W[tl.x];
    if (MK != (w.d_marker != nullptr)) continue;
    const Ctl cs = *w.ctl_src;
    const int tix = tile_y(tl.y) * w.ntx + tile_x(tl.y);
    if (tix == 0 && threadIdx.x == 0) {
      Ctl cd = cs;
      if (cs.remaining > 0) { cd.t += 1; cd.remaining -= 1; }
      *w.ctl_dst = cd;
    }
    if (cs.remaining <= 0) continue;
    const int nx = w.nx, ny = w.ny, ncell = nx * ny;
    const int x0 = tile_x(tl.y) * TILE, y0 = tile_y(tl.y) * TILE;
    const int tw = min(TILE, nx - x0), th = min(TILE, ny - y0);
    const bool append = w.tl_kind != kNoLists && cs.remaining > 1;
    // (the gradient's loads first: they need no other, and loads return in order)
    const WindowLoads<kThreads, kGSide> grad(glbv<const vf2>(w.grad), nx, ny, x0 - LO - (MK ? 4 : 3), y0 - LO - (MK ? 4 : 3));
    SpreadNodes<TILE> nodes(w, tix, glb(w.fel_el));
    zero_lds_u64(s_fx, SW::kCells);
    zero_lds_u64(s_fy, SW::kCells);
    if (append) init_append(w, tile_x(tl.y), tile_y(tl.y), s_app);
    grad.store(s_g);
    // the populations of the tile's cells and those around it, and the nodes
    // to integrate, are on their way while the forces are spread
    const MC_GLOBAL float* src = glb(w.f_src);
    float g[kAhead ? kIt : 1][9];
    const int cx0 = wrap_index(x0 - LO, nx), cy0 = wrap_index(y0 - LO, ny);
    auto load = [&](int i, float* o) {
      const int k = min((int)threadIdx.x + kThreads * i, kCells - 1);
      const int r = k / kStage, c = k - r * kStage;
      const size_t idx = (size_t)wrap_index(cy0 + r, ny) * nx + wrap_index(cx0 + c, nx);
#pragma unroll
      for (int q = 0; q < 9; ++q) o[q] = src[(size_t)q * ncell + idx];
    };
    if constexpr (kAhead) {
#pragma unroll
      for (int i = 0; i < kIt; ++i) load(i, g[i]);
    }
    OwnNodes<TILE> own(w, tix);
    __syncthreads();
    if constexpr (MK)
      tile_spread_markers<TILE, true, LO, HI>(w, nodes, x0, y0, tw, th, 1.0f, s_fx, s_fy, s_g);
    else
      tile_spread_vec<TILE, true, false, LO, HI>(w, nodes, x0, y0, tw, th, 1.0f, s_fx, s_fy, s_g);
    if (__builtin_expect(append && own.L.outgrows, 0)) take_places(w, tile_x(tl.y), tile_y(tl.y), s_app);
    __syncthreads();
    MC_GLOBAL float* dst = glb(w.f_dst);
    // the velocity and the grid force are written where no later step of the
    // call replaces them: on the world's last step, and the velocity on the last
    // of every launched group of steps of a batch, whose worlds can be retired
    // with steps left
    const bool keep_F = w.keep_force || cs.remaining == 1, keep_u = keep || keep_F;
    auto cell = [&](int i, const float* g) {
      const int k = (int)threadIdx.x + kThreads * i;
      if (k >= kCells) return;
      const int r = k / kStage, c = k - r * kStage;
      vf2 F;
      F.x = fix_to_float(spread_cell<SW::kSide>(s_fx, c, r, nx, ny));
      F.y = fix_to_float(spread_cell<SW::kSide>(s_fy, c, r, nx, ny));
      float drho;
      const vf2 u = fluid_velocity(g, F, &drho);
      s_g[k] = u;
      if (c < LO || c >= LO + tw || r < LO || r >= LO + th) return;   // around the tile: the velocity alone
      const int x = x0 + c - LO, y = y0 + r - LO;
      const size_t idx = (size_t)y * nx + x;
      if (keep_u) glbv<vf2>(w.u)[idx] = u;
      if (keep_F) glbv<vf2>(w.Fg)[idx] = F;
      if (!(u.x * u.x + u.y * u.y <= w.u_max2)) atomicOr((unsigned*)glb(w.flags), kFlagUnstable);
      float out[9];
      collide(w, g, F, u, drho, out);
      push(x, y, nx, ny, out, [&](int q, int c, float v) { (dst + (size_t)q * ncell)[c] = v; });
    };
    if constexpr (kAhead) {
#pragma unroll
      for (int i = 0; i < kIt; ++i) cell(i, g[i]);
    } else {
#pragma unroll 1
      for (int i = 0; i < kIt; ++i) {
        load(i, g[0]);
        cell(i, g[0]);
      }
    }
    __syncthreads();
    integrate_own<TILE, MK>(w, own, tl.y, append, s_g, s_app);
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------
// Energy field: every node senses e_i = sum_c W(c - x_i) E_c at the step's
// starting position and collects rate * e_i, which its filament's total
// gains (summed in node order by the filament's first node) and the field
// loses through the same kernel (k_energy_deplete: tile-binned worlds spread
// it over the tile lists in 64-bit fixed point; others with float atomics).
// ---------------------------------------------------------------------------
template <int PACK>
__global__ __launch_bounds__(PACK) void k_energy_gather(const WorldDev* __restrict__ W, Tables T) {
  __shared__ float s_c[PACK];
  __shared__ int s_off[PACK + 1];
  const int npk = *T.n_packs;
  const int li = threadIdx.x;
  for (int it = blockIdx.x; it < npk; it += gridDim.x) {
    const Pack pk = T.packs[it];
    const WorldDev& w = W[pk.world];
    if (!w.energy || w.ctl_src->remaining <= 0) continue;     // block-uniform
    const int N = w.n_part, nx = w.nx, ny = w.ny;
    const int nf = pk.fil_end - pk.fil_begin;
    for (int k = li; k <= nf; k += PACK) s_off[k] = glb(w.fil_offset)[pk.fil_begin + k] - pk.node_begin;
    const int gi = pk.node_begin + li;
    float c = 0.f;
    if (gi < pk.node_end) {
      const int bx = wrap_index(glb(w.cell_in)[gi], nx), by = wrap_index(glb(w.cell_in)[N + gi], ny);
      float wx[4], wy[4];
      peskin4(glb(w.frac_in)[gi], wx);
      peskin4(glb(w.frac_in)[N + gi], wy);
      const MC_GLOBAL float* E = glb(w.energy);
      float e = 0.f;
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        const size_t row = (size_t)wrap_near(by - 1 + b, ny) * nx;
        float a = 0.f;
#pragma unroll
        for (int q = 0; q < 4; ++q) a += wx[q] * E[row + wrap_near(bx - 1 + q, nx)];
        e += wy[b] * a;
      }
      glb(w.e_node)[gi] = e;
      if (w.e_sensed) glb(w.e_sensed)[gi] = e;
      c = w.energy_rate * e;
    }
    s_c[li] = c;
    __syncthreads();
    if (w.e_collected && li < nf) {
      // in node order; the loads eight at a time, so that one lane's chain
      // of adds does not wait for each load in turn
      float sum = 0.f;
      int k = s_off[li];
      const int k1 = s_off[li + 1];
      for (; k + 8 <= k1; k += 8) {
        float v[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) v[q] = s_c[k + q];
#pragma unroll
        for (int q = 0; q < 8; ++q) sum += v[q];
      }
      for (; k < k1; ++k) sum += s_c[k];
      glb(w.e_collected)[pk.fil_begin + li] += sum;
    }
    __syncthreads();
  }
}

template <int TILE>
__global__ __launch_bounds__(TileCfg<TILE>::kThreads) void k_energy_deplete(const WorldDev* __restrict__ W,
                                                                             Tables T) {
  using C = TileCfg<TILE>;
  using SW = SpreadWin<TILE>;
  constexpr int kThreads = C::kThreads;
  __shared__ __align__(16) long long s_x[SW::kCells];
  const int nt = n_tiles<TILE>(T);
  const XcdLoop tiles(nt);
  for (int it = tiles.first; it < tiles.end; it += tiles.step) {
    const int2 tl = tile_entry<TILE>(T, it);
    const WorldDev& w = W[tl.x];
    if (!w.energy || w.mode != kBinned || w.ctl_src->remaining <= 0) continue;
    const int nx = w.nx, ny = w.ny;
    const int x0 = tile_x(tl.y) * TILE, y0 = tile_y(tl.y) * TILE;
    const int tw = min(TILE, nx - x0), th = min(TILE, ny - y0);
    const int tix = tile_y(tl.y) * w.ntx + tile_x(tl.y);
    SpreadNodes<TILE, true> nodes(w, tix, glb(w.e_node));
    zero_lds_u64(s_x, SW::kCells);
    __syncthreads();
    tile_spread_vec<TILE, false, true>(w, nodes, x0, y0, tw, th, -w.energy_rate, s_x, nullptr, nullptr);
    __syncthreads();
    MC_GLOBAL float* E = glb(w.energy);
    for (int k = threadIdx.x; k < TILE * TILE; k += kThreads) {
      const int ly = k >> C::kShift, lx = k & (TILE - 1);
      if (lx >= tw || ly >= th) continue;
      const size_t c = (size_t)(y0 + ly) * nx + x0 + lx;
      E[c] += fix_to_float(spread_cell<SW::kSide>(s_x, lx, ly, nx, ny));
    }
    __syncthreads();
  }
}

template <int PACK>
__global__ __launch_bounds__(PACK) void k_energy_deplete_atomic(const WorldDev* __restrict__ W, Tables T) {
  const int npk = *T.n_packs;
  for (int it = blockIdx.x; it < npk; it += gridDim.x) {
    const Pack pk = T.packs[it];
    const WorldDev& w = W[pk.world];
    if (!w.energy || w.mode == kBinned || w.ctl_src->remaining <= 0) continue;
    const int gi = pk.node_begin + threadIdx.x;
    if (gi >= pk.node_end) continue;
    const int N = w.n_part, nx = w.nx, ny = w.ny;
    const int bx = wrap_index(glb(w.cell_in)[gi], nx), by = wrap_index(glb(w.cell_in)[N + gi], ny);
    float wx[4], wy[4];
    peskin4(glb(w.frac_in)[gi], wx);
    peskin4(glb(w.frac_in)[N + gi], wy);
    const float c = -w.energy_rate * glb(w.e_node)[gi];
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      MC_GLOBAL float* row = glb(w.energy) + (size_t)wrap_near(by - 1 + b, ny) * nx;
#pragma unroll
      for (int q = 0; q < 4; ++q) unsafeAtomicAdd((float*)(row + wrap_near(bx - 1 + q, nx)), c * wx[q] * wy[b]);
    }
  }
}

// Gaussian packets added to a field, every cell (minimum image).
// One block per 32x32 tile: the packets that can reach the tile are listed
// (in index order) and each cell sums only those, in that order.  A packet
// whose nearest distance to the tile (minimum image, less one cell for
// rounding) exceeds sqrt(220) widths has exp(-r^2 / (2 s^2)) below e^-110,
// which is exactly 0 in FP32 (below half the smallest denormal), at every
// cell of the tile, so the sum is the full sum bit for bit.
constexpr int kPacketTile = 32;
constexpr int kPacketChunk = 1024;               // packets listed per pass
__global__ __launch_bounds__(256) void k_energy_packets(int nx, int ny, int n_packets, const float* centres,
                                                        const float* amps, const float* widths, float* field) {
  __shared__ int s_list[kPacketChunk];
  __shared__ int s_wave[4];
  const int ntx = (nx + kPacketTile - 1) / kPacketTile, nty = (ny + kPacketTile - 1) / kPacketTile;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  for (int t = blockIdx.x; t < ntx * nty; t += gridDim.x) {
    const int x0 = (t % ntx) * kPacketTile, y0 = (t / ntx) * kPacketTile;
    const int x1 = min(x0 + kPacketTile, nx) - 1, y1 = min(y0 + kPacketTile, ny) - 1;
    const float hx = 0.5f * (float)(x1 - x0), hy = 0.5f * (float)(y1 - y0);
    const float mx = 0.5f * (float)(x0 + x1), my = 0.5f * (float)(y0 + y1);
    float acc[4] = {0.f, 0.f, 0.f, 0.f};             // cells tid + 256 k of the tile
    for (int p0 = 0; p0 < n_packets; p0 += kPacketChunk) {
      // list this chunk's packets that can reach the tile, in index order:
      // thread tid tests packets p0 + 4 tid .. + 3
      int keep[4];
      int n_keep = 0;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int pi = p0 + 4 * tid + q;
        keep[q] = 0;
        if (pi < n_packets) {
          float dx = centres[pi] - mx, dy = centres[n_packets + pi] - my;
          dx -= (float)nx * floorf(dx / (float)nx + 0.5f);
          dy -= (float)ny * floorf(dy / (float)ny + 0.5f);
          const float ex = fmaxf(fabsf(dx) - hx - 1.0f, 0.f), ey = fmaxf(fabsf(dy) - hy - 1.0f, 0.f);
          const float s = widths[pi];
          keep[q] = ex * ex + ey * ey <= 220.0f * s * s ? 1 : 0;
          n_keep += keep[q];
        }
      }
      // exclusive prefix of n_keep over the block (thread order = packet order)
      int x = n_keep;
#pragma unroll
      for (int off = 1; off < 64; off <<= 1) {
        const int y = __shfl_up(x, off);
        if (lane >= off) x += y;
      }
      if (lane == 63) s_wave[wv] = x;
      __syncthreads();
      int base = x - n_keep;
      for (int j = 0; j < wv; ++j) base += s_wave[j];
      const int total = s_wave[0] + s_wave[1] + s_wave[2] + s_wave[3];
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (keep[q]) s_list[base++] = p0 + 4 * tid + q;
      __syncthreads();
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int c = tid + 256 * k;
        const int x = x0 + (c & (kPacketTile - 1)), y = y0 + (c >> 5);
        if (x > x1 || y > y1) continue;
        float a = acc[k];
        for (int i = 0; i < total; ++i) {
          const int p = s_list[i];
          float dx = (float)x - centres[p], dy = (float)y - centres[n_packets + p];
          dx -= (float)nx * floorf(dx / (float)nx + 0.5f);
          dy -= (float)ny * floorf(dy / (float)ny + 0.5f);
          const float s = widths[p];
          a += amps[p] * expf(-(dx * dx + dy * dy) / (2.0f * s * s));
        }
        acc[k] = a;
      }
      __syncthreads();
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int c = tid + 256 * k;
      const int x = x0 + (c & (kPacketTile - 1)), y = y0 + (c >> 5);
      if (x <= x1 && y <= y1) field[(size_t)y * nx + x] += acc[k];
    }
  }
}

// ---------------------------------------------------------------------------
// Coupling leakage fixes (direct transfer).  Two layers: node i is broadcast
// as markers X = x_i +- d_i, d_i = offset * unit normal (the tangent is
// x_next - x_prev where the node has two neighbours, the edge direction at a
// chain end, none for a lone node).  MDF: desired node velocity
// U_d = I2[j / rho] + F / 2; each further iteration samples
// u = (j + F_grid / 2) / rho at the markers and spreads 2 (U_d - I2[u]).
// ---------------------------------------------------------------------------
template <int PACK>
__global__ __launch_bounds__(PACK) void k_markers(const WorldDev* __restrict__ W, Tables T) {
  __shared__ int s_off[PACK + 1];
  const int npk = *T.n_packs;
  const int li = threadIdx.x;
  for (int it = blockIdx.x; it < npk; it += gridDim.x) {
    const Pack pk = T.packs[it];
    const WorldDev& w = W[pk.world];
    if (!w.d_marker || w.ctl_src->remaining <= 0) continue;     // block-uniform
    const int nf = pk.fil_end - pk.fil_begin;
    for (int k = li; k <= nf; k += PACK) s_off[k] = glb(w.fil_offset)[pk.fil_begin + k] - pk.node_begin;
    __syncthreads();
    const int gi = pk.node_begin + li;
    if (gi < pk.node_end) {
      int lo = 0, hi = nf - 1;
      while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (s_off[mid] <= li) lo = mid; else hi = mid - 1;
      }
      const int o = s_off[lo], n = s_off[lo + 1] - o, k = li - o;
      const int fil = pk.fil_begin + lo;
      const bool ring = w.fil_flags && (glb(w.fil_flags)[fil] & 1) && n >= 3;
      const int first = pk.node_begin + o;
      int a = gi, b = gi;                         // the nodes the tangent joins
      if (k > 0) a = gi - 1; else if (ring) a = first + n - 1;
      if (k < n - 1) b = gi + 1; else if (ring) b = first;
      marker_displacement(w, gi, a, b);
    }
    __syncthreads();
  }
}

// (rho, j) of the step's populations (stored shifted by the weights, whose
// first moment is zero), per cell.
__global__ __launch_bounds__(256) void k_mdf_moments(const WorldDev* __restrict__ W, Tables T) {
  const int nit = *T.n_items;
  for (int it = blockIdx.x; it < nit; it += gridDim.x) {
    const int2 item = T.items[it];
    const WorldDev& w = W[item.x];
    if (w.mdf_iters <= 1 || w.ctl_src->remaining <= 0) continue;
    const int ncell = w.nx * w.ny;
    const int c = item.y + threadIdx.x;
    if (c >= ncell) continue;
    const MC_GLOBAL float* src = glb(w.f_src);
    float g[9];
#pragma unroll
    for (int q = 0; q < 9; ++q) g[q] = src[(size_t)q * ncell + c];
    const float drho = ((g[0] + g[1]) + (g[2] + g[3])) + ((g[4] + g[5]) + (g[6] + g[7])) + g[8];
    const float jx = (g[1] - g[3]) + (g[5] - g[6]) + (g[8] - g[7]);
    const float jy = (g[2] - g[4]) + (g[5] - g[8]) + (g[6] - g[7]);
    const vf4 m = {1.0f + drho, jx, jy, 0.f};
    glbv<vf4>(w.rho_j)[c] = m;
  }
}

// u = (j + F_grid / 2) / rho of the current grid force, per cell.
__global__ __launch_bounds__(256) void k_mdf_velocity(const WorldDev* __restrict__ W, Tables T, int iter) {
  const int nit = *T.n_items;
  for (int it = blockIdx.x; it < nit; it += gridDim.x) {
    const int2 item = T.items[it];
    const WorldDev& w = W[item.x];
    if (w.mode == kBinned || iter >= w.mdf_iters || w.ctl_src->remaining <= 0) continue;
    const int ncell = w.nx * w.ny;
    const int c = item.y + threadIdx.x;
    if (c >= ncell) continue;
    const vf4 m = glbv<const vf4>(w.rho_j)[c];
    const vf2 F = glbv<const vf2>(w.Fg)[c];
    const float inv = 1.0f / m.x;
    const vf2 u = {(m.y + 0.5f * F.x) * inv, (m.z + 0.5f * F.y) * inv};
    glbv<vf2>(w.u_mdf)[c] = u;
  }
}

// Two-layer interpolation of a per-cell quantity at node gi: mean over its
// markers (or the node itself with one layer) of sum_c W(c - X) value(c).
template <class V>
static __device__ __forceinline__ vf2 interp2(const WorldDev& w, int gi, V value) {
  const int N = w.n_part, nx = w.nx, ny = w.ny;
  const int cx = glb(w.cell_in)[gi], cy = glb(w.cell_in)[N + gi];
  const float fx = glb(w.frac_in)[gi], fy = glb(w.frac_in)[N + gi];
  const float dx = w.d_marker ? glb(w.d_marker)[gi] : 0.f, dy = w.d_marker ? glb(w.d_marker)[N + gi] : 0.f;
  float sx = 0.f, sy = 0.f;
  const int layers = w.d_marker ? 2 : 1;
  for (int l = 0; l < layers; ++l) {
    const float sg = l == 0 ? 1.f : -1.f;
    int hx, hy;
    float mx, my;
    marker_home(cx, fx, sg * dx, nx, &hx, &mx);
    marker_home(cy, fy, sg * dy, ny, &hy, &my);
    float wx[4], wy[4];
    peskin4(mx, wx);
    peskin4(my, wy);
    float gx = 0.f, gy = 0.f;
    for (int b = 0; b < 4; ++b) {
      const size_t row = (size_t)wrap_near(hy - 1 + b, ny) * nx;
      float ax = 0.f, ay = 0.f;
      for (int a = 0; a < 4; ++a) {
        const vf2 v = value(row + wrap_near(hx - 1 + a, nx));
        ax += wx[a] * v.x;
        ay += wx[a] * v.y;
      }
      gx += wy[b] * ax;
      gy += wy[b] * ay;
    }
    sx += gx;
    sy += gy;
  }
  const float h = layers == 2 ? 0.5f : 1.0f;
  const vf2 out = {h * sx, h * sy};
  return out;
}

// Spread of (vx, vy) from node gi's markers (half each) or the node.
static __device__ __forceinline__ void spread2_atomic(const WorldDev& w, int gi, float vx, float vy) {
  const int N = w.n_part, nx = w.nx, ny = w.ny;
  const int cx = glb(w.cell_in)[gi], cy = glb(w.cell_in)[N + gi];
  const float fx = glb(w.frac_in)[gi], fy = glb(w.frac_in)[N + gi];
  if (!w.d_marker) {
    atomic_spread_vec(glb((float*)w.Fg), nx, ny, wrap_index(cx, nx), wrap_index(cy, ny), fx, fy, vx, vy);
    return;
  }
  const float dx = glb(w.d_marker)[gi], dy = glb(w.d_marker)[N + gi];
  for (int sg = 1; sg >= -1; sg -= 2) {
    int hx, hy;
    float mx, my;
    marker_home(cx, fx, sg * dx, nx, &hx, &mx);
    marker_home(cy, fy, sg * dy, ny, &hy, &my);
    atomic_spread_vec(glb((float*)w.Fg), nx, ny, hx, hy, mx, my, 0.5f * vx, 0.5f * vy);
  }
}

template <int PACK>
__global__ __launch_bounds__(PACK) void k_mdf_desired(const WorldDev* __restrict__ W, Tables T) {
  const int npk = *T.n_packs;
  for (int it = blockIdx.x; it < npk; it += gridDim.x) {
    const Pack pk = T.packs[it];
    const WorldDev& w = W[pk.world];
    if (w.mode == kBinned || w.mdf_iters <= 1 || w.ctl_src->remaining <= 0) continue;
    const int gi = pk.node_begin + threadIdx.x;
    if (gi >= pk.node_end) continue;
    const MC_GLOBAL vf4* m = glbv<const vf4>(w.rho_j);
    const vf2 us = interp2(w, gi, [&](size_t c) {
      const vf4 v = m[c];
      const vf2 r = {v.y / v.x, v.z / v.x};
      return r;
    });
    const int N = w.n_part;
    glb(w.U_d)[gi] = us.x + 0.5f * glb(w.fel)[gi];
    glb(w.U_d)[N + gi] = us.y + 0.5f * glb(w.fel)[N + gi];
  }
}

template <int PACK>
__global__ __launch_bounds__(PACK) void k_mdf_correct(const WorldDev* __restrict__ W, Tables T, int iter) {
  const int npk = *T.n_packs;
  for (int it = blockIdx.x; it < npk; it += gridDim.x) {
    const Pack pk = T.packs[it];
    const WorldDev& w = W[pk.world];
    if (w.mode == kBinned || iter >= w.mdf_iters || w.ctl_src->remaining <= 0) continue;
    const int gi = pk.node_begin + threadIdx.x;
    if (gi >= pk.node_end) continue;
    const MC_GLOBAL vf2* um = glbv<const vf2>(w.u_mdf);
    const vf2 U = interp2(w, gi, [&](size_t c) { return um[c]; });
    const int N = w.n_part;
    const float cx = 2.0f * (glb(w.U_d)[gi] - U.x);
    const float cy = 2.0f * (glb(w.U_d)[N + gi] - U.y);
    spread2_atomic(w, gi, cx, cy);
  }
}

// Binned transfer: the node passes of MDF as tile passes over the home-tile
// own nodes, and the correction spread through the tiles' lists, summed in
// LDS as 64-bit fixed point like the force spread: deterministic and without
// HBM atomics.
//   k_mdf_gather_tile<TILE, true>   U_d = I[j / rho] + F / 2 at the tile's nodes
//   k_mdf_gather_tile<TILE, false>  c = 2 (U_d - I[(j + F_grid / 2) / rho])
//   k_mdf_spread_tile<TILE>         F_grid += S[c] over the tile
// The velocity is formed per staged cell from the moments and the grid force.
// MK: the two-layer variants (I: the mean over the node's two markers; S:
// half of the value from each marker).
template <int TILE, bool DESIRED, bool MK>
__global__ __launch_bounds__(TileCfg<TILE>::kThreads) void k_mdf_gather_tile(const WorldDev* __restrict__ W, Tables T,
                                                                             int iter) {
  constexpr int kE = MK ? 1 : 0;
  constexpr int kStage = TILE + 3 + 2 * kE, kThreads = TileCfg<TILE>::kThreads;
  constexpr int kIt = (kStage * kStage + kThreads - 1) / kThreads;
  __shared__ vf2 s_u[kStage * kStage];
  const int nt = n_tiles<TILE>(T);
  const XcdLoop tiles(nt);
  for (int it = tiles.first; it < tiles.end; it += tiles.step) {
    const int2 tl = tile_entry<TILE>(T, it);
    const WorldDev& w = W[tl.x];
    if (w.mode != kBinned || w.mdf_iters <= 1 || (!DESIRED && iter >= w.mdf_iters) || w.ctl_src->remaining <= 0)
      continue;
    if (MK != (w.d_marker != nullptr)) continue;
    const int nx = w.nx, ny = w.ny, N = w.n_part;
    const int x0 = tile_x(tl.y) * TILE, y0 = tile_y(tl.y) * TILE;
    const MC_GLOBAL vf4* m = glbv<const vf4>(w.rho_j);
    const MC_GLOBAL vf2* Fg = glbv<const vf2>(w.Fg);
    const int tile = tile_y(tl.y) * w.ntx + tile_x(tl.y);
    vf4 mv[kIt];
    vf2 fv[kIt];
#pragma unroll
    for (int i = 0; i < kIt; ++i) {              // all loads in flight before the stores
      const int k = min((int)threadIdx.x + kThreads * i, kStage * kStage - 1);
      const int r = k / kStage, c = k - (k / kStage) * kStage;
      const size_t idx = (size_t)wrap_index(y0 - 1 - kE + r, ny) * nx + wrap_index(x0 - 1 - kE + c, nx);
      mv[i] = m[idx];
      if (!DESIRED) fv[i] = Fg[idx];
    }
#pragma unroll
    for (int i = 0; i < kIt; ++i) {
      const int k = (int)threadIdx.x + kThreads * i;
      if (k < kStage * kStage) {
        const float inv = 1.0f / mv[i].x;
        vf2 u;
        if (DESIRED) {
          u.x = mv[i].y / mv[i].x;
          u.y = mv[i].z / mv[i].x;
        } else {
          u.x = (mv[i].y + 0.5f * fv[i].x) * inv;
          u.y = (mv[i].z + 0.5f * fv[i].y) * inv;
        }
        s_u[k] = u;
      }
    }
    __syncthreads();
    MC_GLOBAL float* Ud = glb(w.U_d);
    for_own_records<kThreads>(w, tile, x0, y0, min(TILE, nx - x0), min(TILE, ny - y0), [&](const vi4& r) {
      const int lx = (r.x & 0xffff) - x0, ly = (r.x >> 16) - y0;
      const float fx = __int_as_float(r.y), fy = __int_as_float(r.z);
      const int gi = r.w;
      vf2 g;
      if constexpr (MK) {
        g.x = g.y = 0.f;
        const float ddx = glb(w.d_marker)[gi], ddy = glb(w.d_marker)[N + gi];
#pragma unroll
        for (int l = 0; l < 2; ++l) {
          const float sg = l == 0 ? 1.f : -1.f;
          int sx, sy;
          float mx, my;
          marker_shift(fx, sg * ddx, &sx, &mx);
          marker_shift(fy, sg * ddy, &sy, &my);
          float wx[4], wy[4];
          peskin4(mx, wx);
          peskin4(my, wy);
          const vf2 gl = gather_staged<TILE, 1>(s_u, lx + sx + 1, ly + sy + 1, wx, wy);
          g.x += gl.x;
          g.y += gl.y;
        }
        g.x *= 0.5f;
        g.y *= 0.5f;
      } else {
        float wx[4], wy[4];
        peskin4(fx, wx);
        peskin4(fy, wy);
        g = gather_staged<TILE>(s_u, lx, ly, wx, wy);
      }
      if (DESIRED) {
        Ud[gi] = g.x + 0.5f * glb(w.fel)[gi];
        Ud[N + gi] = g.y + 0.5f * glb(w.fel)[N + gi];
      } else {
        glb(w.mdf_c)[gi] = 2.0f * (Ud[gi] - g.x);
        glb(w.mdf_c)[N + gi] = 2.0f * (Ud[N + gi] - g.y);
      }
    });
    __syncthreads();
  }
}

template <int TILE, bool MK>
__global__ __launch_bounds__(TileCfg<TILE>::kThreads) void k_mdf_spread_tile(const WorldDev* __restrict__ W, Tables T,
                                                                             int iter) {
  using C = TileCfg<TILE>;
  using SW = SpreadWin<TILE>;
  constexpr int kThreads = C::kThreads;
  __shared__ __align__(16) long long s_fx[SW::kCells];
  __shared__ __align__(16) long long s_fy[SW::kCells];
  const int nt = n_tiles<TILE>(T);
  const XcdLoop tiles(nt);
  for (int it = tiles.first; it < tiles.end; it += tiles.step) {
    const int2 tl = tile_entry<TILE>(T, it);
    const WorldDev& w = W[tl.x];
    if (w.mode != kBinned || iter >= w.mdf_iters || w.ctl_src->remaining <= 0) continue;
    if (MK != (w.d_marker != nullptr)) continue;
    const int nx = w.nx, ny = w.ny;
    const int x0 = tile_x(tl.y) * TILE, y0 = tile_y(tl.y) * TILE;
    const int tw = min(TILE, nx - x0), th = min(TILE, ny - y0);
    const int tix = tile_y(tl.y) * w.ntx + tile_x(tl.y);
    SpreadNodes<TILE> nodes(w, tix, glb(w.mdf_c));
    zero_lds_u64(s_fx, SW::kCells);
    zero_lds_u64(s_fy, SW::kCells);
    __syncthreads();
    if constexpr (MK)
      tile_spread_markers<TILE, false>(w, nodes, x0, y0, tw, th, 1.0f, s_fx, s_fy, nullptr);
    else
      tile_spread_vec<TILE, false>(w, nodes, x0, y0, tw, th, 1.0f, s_fx, s_fy, nullptr);
    __syncthreads();
    MC_GLOBAL vf2* Fg = glbv<vf2>(w.Fg);
    for (int k = threadIdx.x; k < TILE * TILE; k += kThreads) {
      const int ly = k >> C::kShift, lx = k & (TILE - 1);
      if (lx >= tw || ly >= th) continue;
      const size_t c = (size_t)(y0 + ly) * nx + x0 + lx;
      vf2 F = Fg[c];
      F.x += fix_to_float(spread_cell<SW::kSide>(s_fx, lx, ly, nx, ny));
      F.y += fix_to_float(spread_cell<SW::kSide>(s_fy, lx, ly, nx, ny));
      Fg[c] = F;
    }
    __syncthreads();
  }
}

__global__ void k_set_ctl(Ctl* c, long long t, int remaining) {
  if (threadIdx.x == 0 && blockIdx.x == 0) {
    Ctl v;
    v.t = t;
    v.remaining = remaining;
    v.pad = 0;
    *c = v;
  }
}

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------
#define MC_PACK_DISPATCH(KERNEL, G, ...)                                         \
  do {                                                                           \
    if ((G).pack == 256)                                                         \
      KERNEL<256><<<(G).node_blocks, 256, 0, s>>>(__VA_ARGS__);                  \
    else                                                                         \
      KERNEL<1024><<<(G).node_blocks, 1024, 0, s>>>(__VA_ARGS__);                \
  } while (0)

void launch_elastic(const WorldDev* W, const Tables& T, const Grid& G, hipStream_t s) {
  if (G.branches) {
    if (G.pack == 256)
      k_elastic<256, true, true><<<G.node_blocks, 256, 0, s>>>(W, T);
    else
      k_elastic<1024, true, true><<<G.node_blocks, 1024, 0, s>>>(W, T);
  } else if (G.general) {
    if (G.pack == 256)
      k_elastic<256, true, false><<<G.node_blocks, 256, 0, s>>>(W, T);
    else
      k_elastic<1024, true, false><<<G.node_blocks, 1024, 0, s>>>(W, T);
  } else {
    if (G.pack == 256)
      k_elastic<256, false, false><<<G.node_blocks, 256, 0, s>>>(W, T);
    else
      k_elastic<1024, false, false><<<G.node_blocks, 1024, 0, s>>>(W, T);
  }
}

void launch_list_prepass(const WorldDev* W, const Tables& T, const Grid& G, long long t, int n_steps, hipStream_t s) {
  if (!G.any_lists && n_steps < 0) return;
  k_lists_zero<<<dim3(!G.any_lists ? 1 : G.world_blocks == 1 ? 64 : 8, G.world_blocks), 256, 0, s>>>(W, T, t, n_steps);
  if (!G.any_lists) return;
  const auto build = [&](auto spill) {
    constexpr bool S = decltype(spill)::value;
    if (G.pack == 256) k_lists_build<256, S><<<G.node_blocks, 256, 0, s>>>(W, T, !G.any_spill);
    else k_lists_build<1024, S><<<G.node_blocks, 1024, 0, s>>>(W, T, !G.any_spill);
  };
  build(std::false_type());
  if (!G.any_spill) return;
  k_lists_reserve<<<dim3(G.world_blocks == 1 ? 64 : 4, G.world_blocks), 256, 0, s>>>(W, T);
  build(std::true_type());
}

void launch_sort(const WorldDev* W, const Tables& T, const Grid& G, hipStream_t s) {
  if (G.any_sorted) {
    k_scan_reduce<<<G.scan_blocks, 256, 0, s>>>(W, T);
    k_scan_partials<<<G.world_blocks, 256, 0, s>>>(W, T);
    k_scan_down<<<G.scan_blocks, 256, 0, s>>>(W, T);
    MC_PACK_DISPATCH(k_scatter, G, W, T);
    MC_PACK_DISPATCH(k_segsort, G, W, T);
  }
}

// Tile kernels: one launch per tile family present.
template <int TILE>
static int filter_lds(const Grid& G) {
  return filter_window_bytes<TILE>(G.max_radius) + filter_density_bytes<TILE>(G.max_radius);
}

// the largest dynamic LDS any launch of kernel F asks for (64-cell tiles exceed
// 64 KiB), declared once per kernel and process
template <int TILE, auto F>
static void declare_lds() {
  static const bool done = [] {
    return hipFuncSetAttribute(reinterpret_cast<const void*>(F), hipFuncAttributeMaxDynamicSharedMemorySize,
                               filter_window_bytes<TILE>(kMaxRadius) + filter_density_bytes<TILE>(kMaxRadius)) ==
           hipSuccess;
  }();
  (void)done;
}

template <int TILE>
static void launch_filter_t(const WorldDev* W, const Tables& T, const Grid& G, hipStream_t s) {
  constexpr int f = TileCfg<TILE>::kFamily;
  if (G.tile_blocks[f] <= 0) return;
  if constexpr (TILE == 64) declare_lds<TILE, &k_filter<TILE>>();
  k_filter<TILE><<<G.tile_blocks[f], TileCfg<TILE>::kThreads, filter_lds<TILE>(G), s>>>(
      W, T, filter_window_bytes<TILE>(G.max_radius));
}

void launch_filter(const WorldDev* W, const Tables& T, const Grid& G, hipStream_t s) {
  launch_filter_t<16>(W, T, G, s);
  launch_filter_t<32>(W, T, G, s);
  launch_filter_t<64>(W, T, G, s);
}

template <int TILE, int PACK>
static void launch_prepare_t(const WorldDev* W, const Tables& T, const Grid& G, hipStream_t s) {
  const int tr = (G.tile_blocks[TileCfg<TILE>::kFamily] + 7) / 8, pr = (G.node_blocks + 7) / 8;
  const int wb = filter_window_bytes<TILE>(G.max_radius), lds = filter_lds<TILE>(G);
  const auto go = [&](auto gen, auto br) {
    constexpr bool GN = decltype(gen)::value, B = decltype(br)::value;
    const int bytes = std::max(lds, (int)sizeof(ElasticLds<PACK, B>));
    k_prepare<TILE, PACK, GN, B><<<8 * (tr + pr), PACK, bytes, s>>>(W, T, wb, tr, pr);
  };
  if (G.branches) go(std::true_type(), std::true_type());
  else if (G.general) go(std::true_type(), std::false_type());
  else go(std::false_type(), std::false_type());
}

// One launch where every world is binned and their tiles have one side; else the elastic
// force (which the sorted and direct transfers build on), then the rest.
// Filaments of more than 256 nodes are packed by blocks of 1024 threads, which
// suit a tile ill: up to one block per CU the launch saved counts for more (3000 nodes on
// 128^2, 64 tiles: 27.0 -> 21.5 us per step), past it the separate kernels do
// (200,000 on 1200^2: 68.4 against 90.2).
// Otherwise one launch, except where either role fills the chip for many rounds
// by itself.  One launch and two, us per step: 1,048,623 nodes on 2048^2 (4096
// tiles, 5435 packs) 207.1 and 203.7, 921,663 on 1920^2 (3600 tiles, 4786 packs)
// 207.7 and 204.6, 802,912 on 1792^2 (3136, 4183) 167.3 and 167.4; 589,915 on
// 1536^2 (2304, 3088) 123.9 and 125.1, 524,340 on 2048^2 (4096, 2739) 171.5 and
// 172.3, 262,144 (1358) 155.0 and 158.0, 102,467 on 1280^2 (1600, 534) 59.9 and 64.5.
constexpr int kWideTiles = 256, kMergedBlocks = 3000;
bool prepare_merged(const Grid& G) {
  const int tiles = G.tile_blocks[0] + G.tile_blocks[1];
  return !G.any_node && G.any_binned && (G.tile_blocks[0] > 0) != (G.tile_blocks[1] > 0) &&
         (G.pack == 256 ? std::min(tiles, G.node_blocks) <= kMergedBlocks : tiles <= kWideTiles);
}
void launch_prepare(const WorldDev* W, const Tables& T, const Grid& G, hipStream_t s) {
  if (!prepare_merged(G)) {
    launch_elastic(W, T, G, s);
    launch_sort(W, T, G, s);
    launch_filter(W, T, G, s);
  } else if (G.tile_blocks[0] > 0) {
    if (G.pack == 256) launch_prepare_t<16, 256>(W, T, G, s);
    else launch_prepare_t<16, 1024>(W, T, G, s);
  } else {
    if (G.pack == 256) launch_prepare_t<32, 256>(W, T, G, s);
    else launch_prepare_t<32, 1024>(W, T, G, s);
  }
}

void launch_repulse(const WorldDev* W, const Tables& T, const Grid& G, hipStream_t s) {
  if (G.any_node) MC_PACK_DISPATCH(k_repulse, G, W, T);
  // binned worlds form the repulsion inside k_spread
}

// (tile kernels with a one-layer and a two-layer variant: for_tile_variants)
void launch_spread(const WorldDev* W, const Tables& T, const Grid& G, hipStream_t s) {
  for_tile_variants(G, [&](auto tile, auto mk) {
    constexpr int TL = decltype(tile)::value;
    k_spread<TL, decltype(mk)::value><<<G.tile_blocks[TileCfg<TL>::kFamily], TileCfg<TL>::kThreads, 0, s>>>(W, T);
  });
  if (G.tile_blocks[2] > 0) k_spread<64, false><<<G.tile_blocks[2], TileCfg<64>::kThreads, 0, s>>>(W, T);
}

void launch_fluid_tiles(const WorldDev* W, const Tables& T, const Grid& G, bool keep, hipStream_t s) {
  const auto go = [&](auto tile) {
    constexpr int TL = decltype(tile)::value;
    const int blocks = G.tile_blocks[TileCfg<TL>::kFamily];
    if (blocks == 0) return;
    if (!G.mk_only) k_fluid_tile<TL, false><<<blocks, TileCfg<TL>::kThreads, 0, s>>>(W, T, keep);
    if (G.any_markers) k_fluid_tile<TL, true><<<blocks, TileCfg<TL>::kThreads, 0, s>>>(W, T, keep);
  };
  go(std::integral_constant<int, 16>());
  go(std::integral_constant<int, 32>());
}

void launch_lbm(const WorldDev* W, const Tables& T, const Grid& G, hipStream_t s) {
  k_lbm<<<G.item_blocks, 256, 0, s>>>(W, T);
}

void launch_lbm_timed(const WorldDev* W, const Tables& T, const Grid& G, hipStream_t s, hipEvent_t start,
                      hipEvent_t stop) {
  hipExtLaunchKernelGGL(k_lbm, dim3(G.item_blocks), dim3(256), 0, s, start, stop, 0, W, T);
}

void launch_integrate(const WorldDev* W, const Tables& T, const Grid& G, hipStream_t s) {
  if (G.any_node) MC_PACK_DISPATCH(k_integrate, G, W, T);
  if (G.any_binned) {
    for_tile_variants(G, [&](auto tile, auto mk) {
      constexpr int TL = decltype(tile)::value;
      k_integrate_tile<TL, decltype(mk)::value>
          <<<G.tile_blocks[TileCfg<TL>::kFamily], TileCfg<TL>::kThreads, 0, s>>>(W, T);
    });
  }
}

void launch_markers(const WorldDev* W, const Tables& T, const Grid& G, hipStream_t s) {
  if (G.any_markers) MC_PACK_DISPATCH(k_markers, G, W, T);
}

void launch_mdf_moments(const WorldDev* W, const Tables& T, const Grid& G, hipStream_t s) {
  k_mdf_moments<<<G.item_blocks, 256, 0, s>>>(W, T);
}

void launch_mdf(const WorldDev* W, const Tables& T, const Grid& G, hipStream_t s) {
  if (G.mdf_max <= 1) return;
  k_mdf_moments<<<G.item_blocks, 256, 0, s>>>(W, T);
  if (G.any_node) MC_PACK_DISPATCH(k_mdf_desired, G, W, T);
  if (G.any_binned) {
    for_tile_variants(G, [&](auto tile, auto mk) {
      constexpr int TL = decltype(tile)::value;
      k_mdf_gather_tile<TL, true, decltype(mk)::value>
          <<<G.tile_blocks[TileCfg<TL>::kFamily], TileCfg<TL>::kThreads, 0, s>>>(W, T, 0);
    });
  }
  for (int iter = 1; iter < G.mdf_max; ++iter) {
    if (G.any_node) {
      k_mdf_velocity<<<G.item_blocks, 256, 0, s>>>(W, T, iter);
      MC_PACK_DISPATCH(k_mdf_correct, G, W, T, iter);
    }
    if (G.any_binned) {
      for_tile_variants(G, [&](auto tile, auto mk) {
        constexpr int TL = decltype(tile)::value;
        k_mdf_gather_tile<TL, false, decltype(mk)::value>
            <<<G.tile_blocks[TileCfg<TL>::kFamily], TileCfg<TL>::kThreads, 0, s>>>(W, T, iter);
      });
      for_tile_variants(G, [&](auto tile, auto mk) {
        constexpr int TL = decltype(tile)::value;
        k_mdf_spread_tile<TL, decltype(mk)::value>
            <<<G.tile_blocks[TileCfg<TL>::kFamily], TileCfg<TL>::kThreads, 0, s>>>(W, T, iter);
      });
    }
  }
}

void launch_energy(const WorldDev* W, const Tables& T, const Grid& G, hipStream_t s) {
  if (!G.any_energy) return;
  MC_PACK_DISPATCH(k_energy_gather, G, W, T);
  if (G.any_binned) {
    if (G.tile_blocks[0] > 0) k_energy_deplete<16><<<G.tile_blocks[0], TileCfg<16>::kThreads, 0, s>>>(W, T);
    if (G.tile_blocks[1] > 0) k_energy_deplete<32><<<G.tile_blocks[1], TileCfg<32>::kThreads, 0, s>>>(W, T);
  }
  if (G.any_node) MC_PACK_DISPATCH(k_energy_deplete_atomic, G, W, T);
}

void launch_energy_packets(int nx, int ny, int n_packets, const float* centres, const float* amps,
                           const float* widths, float* field, hipStream_t s) {
  const int nt = ((nx + kPacketTile - 1) / kPacketTile) * ((ny + kPacketTile - 1) / kPacketTile);
  k_energy_packets<<<nt < 8192 ? nt : 8192, 256, 0, s>>>(nx, ny, n_packets, centres, amps, widths, field);
}

void launch_set_ctl(Ctl* c, long long t, int remaining, hipStream_t s) {
  k_set_ctl<<<1, 64, 0, s>>>(c, t, remaining);
}

}  // namespace mc
