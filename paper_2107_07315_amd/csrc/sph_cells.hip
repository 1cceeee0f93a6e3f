// Candidate-list build.
//
// The paper's sums run over "particles within the support radius" (section "Solid SPH
// Equations"); with support h_a + h_b the neighbour set is
//   N(a) = { b != a : |x_a - x_b|^2 < (h_a + h_b)^2 }.
// The particle arrays are kept along a global Morton curve and cut into tiles of at most 64
// consecutive particles.  Neighbours are found through bounding boxes over that order: one box per
// 8 consecutive particles of a tile, one per tile, one per 64 tiles, each with its largest h, so a
// search adapts to the tenfold range of smoothing lengths by itself (no grid, no second sort).
// k_build_tiles descends the boxes for every tile and tests what is left on the matrix cores.  FP32
// runs and shells take the lists of a cell grid instead (sph_cellgrid.hip, which says why), and so do very
// large sets (kBoxesMost) and those with a wide skin (wide_skin).
#include <stddef.h>
#include <string.h>

#include <mutex>

#include "sph_build.h"
#include "sph_internal.h"

namespace {

constexpr int kB = 256;

__device__ __forceinline__ unsigned long long wave_min_u64(unsigned long long v) {
  for (int off = 32; off > 0; off >>= 1) {
    unsigned long long o = __shfl_xor(v, off, 64);
    v = o < v ? o : v;
  }
  return v;
}
__device__ __forceinline__ unsigned long long wave_max_u64(unsigned long long v) {
  for (int off = 32; off > 0; off >>= 1) {
    unsigned long long o = __shfl_xor(v, off, 64);
    v = o > v ? o : v;
  }
  return v;
}

// Bounding box and h range: one partial per block (8 encoded values), reduced in set-up.
__global__ __launch_bounds__(kB) void k_bounds(const double* __restrict__ x, const double* __restrict__ y,
                                               const double* __restrict__ z, const double* __restrict__ h, int64_t n,
                                               unsigned long long* __restrict__ partial) {
  __shared__ unsigned long long red[4][8];
  unsigned long long v[8] = {~0ull, ~0ull, ~0ull, 0ull, 0ull, 0ull, ~0ull, 0ull};  // lo xyz, hi xyz, hmin, hmax
  for (int64_t a = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; a < n;
       a += (int64_t)gridDim.x * blockDim.x) {
    double q[3] = {x[a], y[a], z[a]};
    for (int d = 0; d < 3; ++d) {
      unsigned long long e = enc_double(q[d]);
      v[d] = e < v[d] ? e : v[d];
      v[3 + d] = e > v[3 + d] ? e : v[3 + d];
    }
    unsigned long long e = enc_double(h[a]);
    v[6] = e < v[6] ? e : v[6];
    v[7] = e > v[7] ? e : v[7];
  }
  for (int k = 0; k < 8; ++k) {
    bool mx = (k >= 3 && k < 6) || k == 7;
    v[k] = mx ? wave_max_u64(v[k]) : wave_min_u64(v[k]);
  }
  const int wave = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0)
    for (int k = 0; k < 8; ++k) red[wave][k] = v[k];
  __syncthreads();
  if (threadIdx.x < 8) {
    int k = threadIdx.x;
    bool mx = (k >= 3 && k < 6) || k == 7;
    unsigned long long r = red[0][k];
    for (int w = 1; w < 4; ++w) r = mx ? (red[w][k] > r ? red[w][k] : r) : (red[w][k] < r ? red[w][k] : r);
    partial[(int64_t)blockIdx.x * 8 + k] = r;
  }
}

__global__ __launch_bounds__(64) void k_grid_setup1(GridInfo* g, const unsigned long long* __restrict__ partial,
                                                    int nblocks, int periodic, double box, double skin,
                                                    DevStatus* st) {
  unsigned long long v[8] = {~0ull, ~0ull, ~0ull, 0ull, 0ull, 0ull, ~0ull, 0ull};
  for (int b = threadIdx.x; b < nblocks; b += 64)
    for (int k = 0; k < 8; ++k) {
      unsigned long long e = partial[(int64_t)b * 8 + k];
      bool mx = (k >= 3 && k < 6) || k == 7;
      v[k] = mx ? (e > v[k] ? e : v[k]) : (e < v[k] ? e : v[k]);
    }
  for (int k = 0; k < 8; ++k) {
    bool mx = (k >= 3 && k < 6) || k == 7;
    v[k] = mx ? wave_max_u64(v[k]) : wave_min_u64(v[k]);
  }
  if (threadIdx.x != 0) return;
  for (int d = 0; d < 3; ++d) { g->enc_lo[d] = v[d]; g->enc_hi[d] = v[3 + d]; }
  g->enc_hmin = v[6];
  g->enc_hmax = v[7];
  for (int l = 0; l < SPH_MAX_LEV; ++l) {
    g->hlev_bits[l] = 0ull;
    for (int d = 0; d < 3; ++d) {
      g->lev_lo[l][d] = ~0ull;
      g->lev_hi[l][d] = 0ull;
    }
  }
  g->periodic = periodic;
  g->box = box;
  for (int d = 0; d < 3; ++d) g->lo[d] = periodic ? 0.0 : dec_double(g->enc_lo[d]);
  g->hmin = dec_double(g->enc_hmin);
  g->hmax = dec_double(g->enc_hmax);
  // minimum image needs h_a + h_b < box / 2 for every pair; non-positive h is invalid
  if ((periodic && !(2.0 * g->hmax < 0.5 * box)) || !(g->hmin > 0.0)) latch_error(st, SPH_E_ARG, -1);
  // effective skin: the widened support must stay below half a periodic box
  double s = skin;
  if (periodic) {
    const double smax = 0.5 * box / (2.0 * g->hmax) * (1.0 - 1e-9) - 1.0;
    s = s < smax ? s : smax;
  }
  g->skin = s >= 1e-4 ? s : 0.0;
  int L = 1;
  while (L < SPH_MAX_LEV && g->hmax >= g->hmin * (double)(1 << L)) ++L;
  g->nlev = L;
  // origin of the FP32 bounding boxes; a set wider than 2^32 smallest smoothing lengths is refused
  for (int d = 0; d < 3; ++d) g->org[d] = isfinite(g->lo[d]) ? g->lo[d] : 0.0;
  const bool usual = g->hmin > 1e-290 && g->hmin < 1e290;
  g->bunit = usual ? ldexp(1.0, -31 - ilogb(g->hmin)) : 1.0;
  if (!periodic)
    for (int d = 0; d < 3; ++d) {
      const double ext = dec_double(g->enc_hi[d]) - g->lo[d];
      if (ext > 0x1p32 * g->hmin) latch_error(st, SPH_E_ARG, -1);
    }
}

// Reorders the particle arrays: a gather along the permutation into a staging area and a copy back,
// every array of a batch in one launch each (the permutation is read once per particle, and a list
// build at 20k particles is a chain of short launches: one pair instead of six took 40 us off it).
// elem: bytes per element (8, 4 or 1).  crust: an array of type-1 particles only (S, dS/dt), which is 0
// for the others: their old values are not read.
constexpr int kPermMax = 48;
struct PermBatch {
  void* arr[kPermMax];
  char* stage[kPermMax];
  uint8_t elem[kPermMax], crust[kPermMax], back[kPermMax];   // back: copied back from the staging area
  int na;
  const int8_t* type;       // before the permutation
};
__global__ __launch_bounds__(kB) void k_permute_gather(PermBatch B, const uint32_t* __restrict__ perm, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const int64_t j = (int64_t)perm[i];
  const bool crust = B.type[j] == 1;
  for (int k = 0; k < B.na; ++k) {
    if (B.elem[k] == 8)
      reinterpret_cast<double*>(B.stage[k])[i] =
          B.crust[k] && !crust ? 0.0 : reinterpret_cast<const double*>(B.arr[k])[j];
    else if (B.elem[k] == 4)
      reinterpret_cast<int32_t*>(B.stage[k])[i] = reinterpret_cast<const int32_t*>(B.arr[k])[j];
    else
      reinterpret_cast<int8_t*>(B.stage[k])[i] = reinterpret_cast<const int8_t*>(B.arr[k])[j];
  }
}
__global__ __launch_bounds__(kB) void k_permute_copy(PermBatch B, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  for (int k = 0; k < B.na; ++k) {
    if (!B.back[k]) continue;
    if (B.elem[k] == 8)
      reinterpret_cast<double*>(B.arr[k])[i] = reinterpret_cast<const double*>(B.stage[k])[i];
    else if (B.elem[k] == 4)
      reinterpret_cast<int32_t*>(B.arr[k])[i] = reinterpret_cast<const int32_t*>(B.stage[k])[i];
    else
      reinterpret_cast<int8_t*>(B.arr[k])[i] = reinterpret_cast<const int8_t*>(B.stage[k])[i];
  }
}

// pos4: absolute position and h (FP64 pair passes); pos4f: position relative to the
// particle's star centre and h (FP32 pair passes keep full precision near each star).
// After a reordering (pos_build != nullptr) it also keeps the positions and h of the build for the
// skin test and clears the stress rates of the particles that are not of type 1.
__global__ __launch_bounds__(kB) void k_pack_pos(const double* __restrict__ x, const double* __restrict__ y,
                                                 const double* __restrict__ z, const double* __restrict__ h,
                                                 const int32_t* __restrict__ star,
                                                 const StarInfo* __restrict__ stars, int64_t n,
                                                 double4* __restrict__ pos4, float4* __restrict__ pos4f,
                                                 double4* __restrict__ pos_build, const int8_t* __restrict__ type,
                                                 double* __restrict__ dSdt, double* __restrict__ sdot) {
  int64_t a = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (a >= n) return;
  double cx = 0, cy = 0, cz = 0;
  if (pos4f && star && stars) {
    StarInfo s = stars[star[a]];
    cx = s.cx; cy = s.cy; cz = s.cz;
  }
  const double4 q = make_double4(x[a], y[a], z[a], h[a]);
  pos4[a] = q;
  if (pos4f) pos4f[a] = make_float4((float)(q.x - cx), (float)(q.y - cy), (float)(q.z - cz), (float)(0.5 * q.w));
  if (pos_build) {
    pos_build[a] = q;
    if (type[a] != 1) {
      for (int c = 0; c < 6; ++c) dSdt[c * n + a] = 0.0;
      sdot[a] = 0.0;
    }
  }
}

// Global Morton key of a 1024^3 grid over the bounding box: the particle arrays are kept in this
// order (re-sorted every few steps), so any 64 consecutive particles form a compact tile whatever
// the local density.
__global__ __launch_bounds__(kB) void k_gkeys(const double* __restrict__ x, const double* __restrict__ y,
                                              const double* __restrict__ z, int64_t n,
                                              const GridInfo* __restrict__ gp, uint32_t* __restrict__ keys,
                                              uint32_t* __restrict__ vals) {
  const int64_t a = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (a >= n) return;
  const GridInfo& g = *gp;
  double ext = 0.0;
  for (int d = 0; d < 3; ++d) {
    const double e = g.periodic ? g.box : dec_double(g.enc_hi[d]) - g.lo[d];
    ext = e > ext ? e : ext;
  }
  const double sc = ext > 0.0 ? 1024.0 / ext : 0.0;
  uint32_t k3[3];
  const double q[3] = {x[a], y[a], z[a]};
  for (int d = 0; d < 3; ++d) {
    int k = (int)floor((q[d] - g.lo[d]) * sc);
    k3[d] = (uint32_t)(k < 0 ? 0 : (k > 1023 ? 1023 : k));
  }
  keys[a] = spread3(k3[0]) | (spread3(k3[1]) << 1) | (spread3(k3[2]) << 2);
  vals[a] = (uint32_t)a;
}

// Tile table, rebuilt at every full re-sort (particles keep their array order in between).  A
// tile starts at every multiple of 64 and wherever the Morton curve jumps: if consecutive keys first
// differ in octree level k, the two particles only share a block of 2^(k+1) fine cells, so a tile
// that spans the boundary could be that large.  Cutting where 2^(k+1) fine cells exceed 4 h keeps
// every tile inside a region about 4 smoothing lengths across, in dense and sparse parts alike
// (the factor is the tile_cut parameter).
__device__ __forceinline__ double curve_cell(const GridInfo& g) {   // the width of the curve's finest cells
  double ext = 0.0;
  for (int d = 0; d < 3; ++d) {
    const double e = g.periodic ? g.box : dec_double(g.enc_hi[d]) - g.lo[d];
    ext = e > ext ? e : ext;
  }
  return ext / 1024.0;
}
__device__ __forceinline__ double morton_jump(const GridInfo& g, const uint32_t* __restrict__ gkeys, int64_t p) {
  const uint32_t x = gkeys[p] ^ gkeys[p - 1];
  const int lvl = x ? (31 - __clz(x)) / 3 : -1;
  return lvl >= 0 ? (double)(2 << lvl) * curve_cell(g) : 0.0;
}
// Block-wide sums and exclusive scans over 1024 elements a block, 4 consecutive ones a thread
// (256 threads): a count per block, scanned by k_scan_rows, then each element's index.
__device__ __forceinline__ uint32_t wave_inclusive_scan(uint32_t v) {
  const int lane = threadIdx.x & 63;
  for (int off = 1; off < 64; off <<= 1) {
    const uint32_t o = __shfl_up(v, off, 64);
    if (lane >= off) v += o;
  }
  return v;
}
__device__ __forceinline__ uint32_t block_exclusive(uint32_t v, uint32_t& total) {
  __shared__ uint32_t wsum[4];
  const int wave = threadIdx.x >> 6;
  const uint32_t inc = wave_inclusive_scan(v);
  __syncthreads();
  if ((threadIdx.x & 63) == 63) wsum[wave] = inc;
  __syncthreads();
  uint32_t before = 0;
  for (int w = 0; w < wave; ++w) before += wsum[w];
  total = wsum[0] + wsum[1] + wsum[2] + wsum[3];
  return before + inc - v;
}

// The box search of a tile looks at every run of 64 tiles, so its time grows with the square of the set;
// larger FP64 sets take the cell grid's lists.  List build with boxes and with the grid, ms: particles
// spread evenly, 4M 4.0 and 4.0, 8M 8.3 and 8.1, 12M 14.2 and 11.8, 16M 20.4 and 15.4; star of 4M 4.7 and
// 5.2, of 8M 9.5 and 10.4.
constexpr int64_t kBoxesMost = int64_t(1) << 23;

// Start flags of the first cut, and their count per block.
__global__ __launch_bounds__(kB) void k_tile_flags(const uint32_t* __restrict__ gkeys, const double* __restrict__ h,
                                                   int64_t n, const GridInfo* __restrict__ gp, double cut, int len,
                                                   uint32_t* __restrict__ flag, uint32_t* __restrict__ bsum) {
  const int64_t p0 = (int64_t)blockIdx.x * 1024 + threadIdx.x * 4;
  uint32_t v = 0u;
  for (int k = 0; k < 4; ++k) {
    const int64_t p = p0 + k;
    if (p >= n) break;
    const uint32_t f = ((p & (len - 1)) == 0 || morton_jump(*gp, gkeys, p) > cut * h[p]) ? 1u : 0u;
    flag[p] = f;
    v += f;
  }
  uint32_t tot;
  block_exclusive(v, tot);
  if (threadIdx.x == 0) bsum[blockIdx.x] = tot;
}

// The index of each particle's flag (tiles started before it) and the tiles' first particles.
__global__ __launch_bounds__(kB) void k_tile_starts(const uint32_t* __restrict__ flag, const uint32_t* __restrict__ boff,
                                                    int64_t n, uint32_t* __restrict__ idx,
                                                    int32_t* __restrict__ tile_start) {
  const int64_t p0 = (int64_t)blockIdx.x * 1024 + threadIdx.x * 4;
  uint32_t f[4], v = 0u, tot;
  for (int k = 0; k < 4; ++k) {
    f[k] = p0 + k < n ? flag[p0 + k] : 0u;
    v += f[k];
  }
  uint32_t e = block_exclusive(v, tot) + boff[blockIdx.x];
  for (int k = 0; k < 4; ++k) {
    if (p0 + k >= n) break;
    idx[p0 + k] = e;
    if (f[k]) tile_start[e] = (int32_t)(p0 + k);
    e += f[k];
  }
}

__device__ __forceinline__ int32_t tile_length(const int32_t* __restrict__ tile_start, int64_t t, int64_t nt, int64_t n) {
  return (int32_t)((t + 1 < nt ? (int64_t)tile_start[t + 1] : n) - tile_start[t]);
}
// tile lengths alone (the cell grid's first cut)
__global__ __launch_bounds__(kB) void k_tile_len(const GridInfo* __restrict__ gp, int64_t n,
                                                 const int32_t* __restrict__ tile_start, int32_t* __restrict__ tile_cnt) {
  const int64_t nt = gp->ntiles;
  for (int64_t t = (int64_t)blockIdx.x * kB + threadIdx.x; t < nt; t += (int64_t)gridDim.x * kB)
    tile_cnt[t] = tile_length(tile_start, t, nt, n);
}

// The final tiles: each one's reservation in the union pool, min(ucap, cnt * cap) entries, and
// whether it holds a particle of type 1 (crust).  Those tiles are the stress pass's work list:
// breaking only removes particles from the stressed set and type never changes, so the list stays a
// superset until the next build.  Every other particle is of type 0, carries no deviatoric stress and
// has zero stress rates, set once per build (the kicks then skip the stress arrays of type-0
// particles; the rates of type-1 particles are written by the pass).
// One wave a tile finds the type, then both are summed and scanned 1024 tiles a block.
__global__ __launch_bounds__(256) void k_tile_crust(const GridInfo* __restrict__ gp, int64_t n,
                                                    const int32_t* __restrict__ tile_start,
                                                    const int8_t* __restrict__ type, int32_t* __restrict__ tile_cnt,
                                                    uint32_t* __restrict__ crust) {
  const int64_t nt = gp->ntiles;
  const int lane = threadIdx.x & 63;
  for (int64_t t = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); t < nt; t += (int64_t)gridDim.x * 4) {
    const int32_t cnt = tile_length(tile_start, t, nt, n);
    const unsigned long long m = __ballot(lane < cnt && type[tile_start[t] + lane] == 1);
    if (lane == 0) {
      tile_cnt[t] = cnt;
      crust[t] = m ? 1u : 0u;
    }
  }
}
__device__ __forceinline__ uint32_t pool_share(int32_t cnt, int cap, int ucap) {
  const int64_t b = (int64_t)cnt * cap;
  return (uint32_t)(b < ucap ? b : ucap);
}
__global__ __launch_bounds__(kB) void k_tile_sums(const GridInfo* __restrict__ gp, const int32_t* __restrict__ tile_cnt,
                                                  const uint32_t* __restrict__ crust, int cap, int ucap,
                                                  uint32_t* __restrict__ bsum, int nb) {
  const int64_t nt = gp->ntiles, t0 = (int64_t)blockIdx.x * 1024 + threadIdx.x * 4;
  uint32_t u = 0u, c = 0u, tot;
  for (int k = 0; k < 4; ++k)
    if (t0 + k < nt) {
      u += pool_share(tile_cnt[t0 + k], cap, ucap);
      c += crust[t0 + k];
    }
  block_exclusive(u, tot);
  if (threadIdx.x == 0) bsum[blockIdx.x] = tot;
  block_exclusive(c, tot);
  if (threadIdx.x == 0) bsum[nb + blockIdx.x] = tot;
}
__global__ __launch_bounds__(kB) void k_tile_offsets(const GridInfo* __restrict__ gp, const int32_t* __restrict__ tile_cnt,
                                                     const uint32_t* __restrict__ crust, int cap, int ucap,
                                                     const uint32_t* __restrict__ boff, int nb,
                                                     uint32_t* __restrict__ uoff, int32_t* __restrict__ list) {
  const int64_t nt = gp->ntiles, t0 = (int64_t)blockIdx.x * 1024 + threadIdx.x * 4;
  uint32_t u[4], c[4], su = 0u, sc = 0u, tot;
  for (int k = 0; k < 4; ++k) {
    u[k] = t0 + k < nt ? pool_share(tile_cnt[t0 + k], cap, ucap) : 0u;
    c[k] = t0 + k < nt ? crust[t0 + k] : 0u;
    su += u[k];
    sc += c[k];
  }
  uint32_t eu = block_exclusive(su, tot) + boff[blockIdx.x], ec = block_exclusive(sc, tot) + boff[nb + blockIdx.x];
  for (int k = 0; k < 4; ++k) {
    if (t0 + k >= nt) break;
    uoff[t0 + k] = eu;
    eu += u[k];
    if (c[k]) list[ec++] = (int32_t)(t0 + k);
  }
}
// Per tile: whether one of its particles or of its union members is of type 1 (one wave a tile).
__global__ __launch_bounds__(64) void k_tile_union_type(const GridInfo* __restrict__ gp, const int32_t* __restrict__ tile_start,
                                                       const int32_t* __restrict__ tile_cnt,
                                                       const uint32_t* __restrict__ tile_uoff,
                                                       const int32_t* __restrict__ tile_usize,
                                                       const int32_t* __restrict__ tile_u,
                                                       const int8_t* __restrict__ type, uint32_t* __restrict__ flag) {
  const int lane = threadIdx.x;
  const int64_t nt = gp->ntiles;
  for (int64_t t = blockIdx.x; t < nt; t += gridDim.x) {
    bool f = lane < tile_cnt[t] && type[tile_start[t] + lane] == 1;
    const int32_t us = tile_usize[t];
    const int32_t* U = tile_u + tile_uoff[t];
    for (int j = lane; j < us && !f; j += 64) f = type[U[j]] == 1;
    const unsigned long long m = __ballot(f);
    if (lane == 0) flag[t] = m ? 1u : 0u;
  }
}
// ---- bounding boxes ----------------------------------------------------------------------------
__device__ __forceinline__ double wave_min_d(double v) {
  for (int off = 32; off > 0; off >>= 1) v = fmin(v, __shfl_xor(v, off, 64));
  return v;
}
// min / max over aligned groups of NL lanes
template <int NL>
__device__ __forceinline__ double grp_min(double v) {
  for (int off = 1; off < NL; off <<= 1) v = fmin(v, __shfl_xor(v, off, 64));
  return v;
}
template <int NL>
__device__ __forceinline__ double grp_max(double v) {
  for (int off = 1; off < NL; off <<= 1) v = fmax(v, __shfl_xor(v, off, 64));
  return v;
}
__device__ __forceinline__ float round_up(double v) { return (float)v * (1.0f + 0x1p-21f) + 1e-37f; }

// Box of the NL lanes of a group: q = position relative to the origin, h (both in the boxes' unit), in = the
// lane holds a particle with finite values.  The half-width is taken about the FP32-rounded centre and rounded
// up, so the box holds every particle exactly.
template <int NL>
__device__ __forceinline__ Box group_box(const double q[3], double h, bool in) {
  Box B;
  const double big = 1e300;
  float c[3], w[3];
  const bool any = grp_max<NL>(in ? 1.0 : 0.0) > 0.0;
  for (int d = 0; d < 3; ++d) {
    const double lo = grp_min<NL>(in ? q[d] : big), hi = grp_max<NL>(in ? q[d] : -big);
    c[d] = any ? (float)(0.5 * (lo + hi)) : 0.f;
    w[d] = any ? round_up(fmax(hi - (double)c[d], (double)c[d] - lo)) : 0.f;
  }
  const float hm = any ? round_up(grp_max<NL>(in ? h : 0.0)) : -1.f;
  B.c = make_float4(c[0], c[1], c[2], hm);
  B.w = make_float4(w[0], w[1], w[2], 0.f);
  return B;
}

// Whether particles of the two boxes can lie within (h_a + h_b) s1 of each other (s1 widened by
// 1e-5, far above the FP32 rounding of the test; with a periodic box the centres' distance is the
// minimum image, itself widened by its rounding).
template <bool PER>
__device__ __forceinline__ bool boxes_near(const float4& ac, const float4& aw, const float4& bc, const float4& bw,
                                           float s1, float box) {
  float dx = fabsf(ac.x - bc.x), dy = fabsf(ac.y - bc.y), dz = fabsf(ac.z - bc.z);
  if constexpr (PER) {
    const float e = box * 0x1p-21f;
    dx = fminf(dx, box - dx) - e;
    dy = fminf(dy, box - dy) - e;
    dz = fminf(dz, box - dz) - e;
  }
  const float gx = fmaxf(0.f, dx - (aw.x + bw.x)), gy = fmaxf(0.f, dy - (aw.y + bw.y)), gz = fmaxf(0.f, dz - (aw.z + bw.z));
  const float R = (ac.w + bc.w) * s1;
  return gx * gx + gy * gy + gz * gz < R * R && bc.w > 0.f;
}

// Boxes of each tile and of its runs of 8 particles, and what k_tile_crust finds (one wave a tile).
__global__ __launch_bounds__(64) void k_tile_boxes(const GridInfo* __restrict__ gp, const double4* __restrict__ pos4,
                                                   int64_t n, const int32_t* __restrict__ tile_start,
                                                   const int8_t* __restrict__ type, int32_t* __restrict__ tile_cnt,
                                                   uint32_t* __restrict__ crust, Box* __restrict__ tile_box,
                                                   Box* __restrict__ sub_box) {
  const int lane = threadIdx.x;
  const GridInfo& g = *gp;
  const int64_t ntiles = g.ntiles;
  for (int64_t t = blockIdx.x; t < ntiles; t += gridDim.x) {
    const int32_t ts = tile_start[t], tc = tile_length(tile_start, t, ntiles, n);
    const unsigned long long cm = __ballot(lane < tc && type[ts + lane] == 1);
    if (lane == 0) {
      tile_cnt[t] = tc;
      crust[t] = cm ? 1u : 0u;
    }
    const double4 p = lane < tc ? pos4[ts + lane] : make_double4(0.0, 0.0, 0.0, 0.0);
    const double q[3] = {(p.x - g.org[0]) * g.bunit, (p.y - g.org[1]) * g.bunit, (p.z - g.org[2]) * g.bunit};
    const double h = p.w * g.bunit;
    const bool in = lane < tc && isfinite(q[0]) && isfinite(q[1]) && isfinite(q[2]) && isfinite(h);
    const Box sb = group_box<8>(q, h, in), tb = group_box<64>(q, h, in);
    if ((lane & 7) == 0 && lane < tc) sub_box[(ts >> 3) + t + (lane >> 3)] = sb;
    if (lane == 0) tile_box[t] = tb;
  }
}

// Box of each run of 64 tiles (one wave a run).
__global__ __launch_bounds__(64) void k_super_boxes(const GridInfo* __restrict__ gp, const Box* __restrict__ tile_box,
                                                    Box* __restrict__ super_box) {
  const int lane = threadIdx.x;
  const int64_t ntiles = gp->ntiles, ns = (ntiles + 63) / 64;
  for (int64_t s = blockIdx.x; s < ns; s += gridDim.x) {
    const int64_t t = s * 64 + lane;
    Box b;
    b.c.w = -1.f;
    if (t < ntiles) b = tile_box[t];
    const bool in = b.c.w > 0.f;
    // the union of the tiles' boxes, in FP64 from their FP32 corners
    const float bc[3] = {b.c.x, b.c.y, b.c.z}, bw[3] = {b.w.x, b.w.y, b.w.z};
    float c[3], w[3];
    const bool any = __ballot(in) != 0ull;
    for (int d = 0; d < 3; ++d) {
      const double lo = grp_min<64>(in ? (double)bc[d] - (double)bw[d] : 1e300);
      const double hi = grp_max<64>(in ? (double)bc[d] + (double)bw[d] : -1e300);
      c[d] = any ? (float)(0.5 * (lo + hi)) : 0.f;
      w[d] = any ? round_up(fmax(hi - (double)c[d], (double)c[d] - lo)) : 0.f;
    }
    const float hm = (float)grp_max<64>(in ? (double)b.c.w : -1.0);
    if (lane == 0) super_box[s] = Box{make_float4(c[0], c[1], c[2], hm), make_float4(w[0], w[1], w[2], 0.f)};
  }
}

// Cost estimate of each tile: the particles of the tiles near it.
template <bool PER>
__global__ __launch_bounds__(64) void k_tile_cost(const GridInfo* __restrict__ gp, const int32_t* __restrict__ tile_cnt,
                                                  const Box* __restrict__ tile_box, const Box* __restrict__ super_box,
                                                  int32_t* __restrict__ cost) {
  const int lane = threadIdx.x;
  const GridInfo& g = *gp;
  const float s1 = (float)(1.0 + g.skin) * (1.0f + 1e-5f), box = (float)(g.box * g.bunit);
  const int64_t ntiles = g.ntiles, ns = (ntiles + 63) / 64;
  for (int64_t k_ = blockIdx.x / SPH_XCD, chunk_ = xcd_chunk(ntiles); k_ < chunk_; k_ += gridDim.x / SPH_XCD) {
    const int64_t t = (int64_t)(blockIdx.x % SPH_XCD) * chunk_ + k_;
    if (t >= ntiles) break;
    const Box own = tile_box[t];
    int64_t tot = 0;
    for (int64_t s0 = 0; s0 < ns; s0 += 64) {
      bool near = false;
      if (s0 + lane < ns) {
        const Box b = super_box[s0 + lane];
        near = boxes_near<PER>(own.c, own.w, b.c, b.w, s1, box);
      }
      unsigned long long m = __ballot(near);
      while (m) {
        const int64_t u = (s0 + __builtin_ctzll(m)) * 64 + lane;
        m &= m - 1;
        if (u < ntiles) {
          const Box b = tile_box[u];
          if (boxes_near<PER>(own.c, own.w, b.c, b.w, s1, box)) tot += tile_cnt[u];
        }
      }
    }
    for (int off = 32; off > 0; off >>= 1) tot += __shfl_xor(tot, off, 64);
    if (lane == 0) cost[t] = (int32_t)(tot < 0x7fffffff ? tot : 0x7fffffff);
  }
}

// Splits expensive tiles: a particle also starts a tile where the curve jumps farther than 4 (cost >
// kSplit4) or 2 (cost > kSplit2) of the smaller smoothing lengths at the jump, and at every 32nd
// position of the dearer ones.  A tile that spans such a jump near the surface, where h varies
// tenfold, is wide against its smallest h and would test thousands of runs in one wave, which the
// whole build then waits for.  On the 1M-particle star (mean cost 5700) 16.6k tiles become 18.1k
// and the dearest tests 107 batches of 64 candidates (2700 without the split; 36 on average);
// cutting every tile above 8000 at 4 h costs 15% more tiles, which the pair passes pay for at
// every evaluation.  Sets of at most kSplitSmall particles (1100 tiles, about one a SIMD) take half
// the thresholds, sets of kTiles32 a third (their tiles are smaller): there more tiles run side by side, and
// the dearest tile is the build's time.  Where the curve is blind (a cell of it wider than 2 smoothing
// lengths, in a set with particles far outside) the particles of a cell lie in no order, and 32 of them can
// have more candidates between them than a union takes: a tile of such particles is cut so that 1.5 times
// the candidates it can expect (its cost, spread evenly over its box) fit.  100k particles in a cube in no
// order, one more at 1e5 of its sizes, ms an evaluation: cut at every 32nd position 6.0, at every 8th 15.7
// (9.3 with the cell grid's lists, always cut at every 8th; 0.6 without the far particle).
// Reads the tile of p from the scan of the old flags.
constexpr int32_t kSplit4 = 12000, kSplit2 = 18000, kSplitSmall = 65536;
__global__ __launch_bounds__(kB) void k_tile_split(uint32_t* __restrict__ flag, const uint32_t* __restrict__ idx,
                                                   int64_t n, const int32_t* __restrict__ tile_start,
                                                   const int32_t* __restrict__ cost, const uint32_t* __restrict__ gkeys,
                                                   const double4* __restrict__ pos4, const Box* __restrict__ tile_box,
                                                   int ucap, const GridInfo* __restrict__ gp, uint32_t* __restrict__ bsum) {
  const int64_t p0 = (int64_t)blockIdx.x * 1024 + threadIdx.x * 4;
  const int32_t part = n <= kTiles32 ? 3 : (n <= kSplitSmall ? 2 : 1);
  uint32_t v = 0u, tot;
  for (int k = 0; k < 4; ++k) {
    const int64_t p = p0 + k;
    if (p >= n) break;
    bool f = flag[p] != 0u;
    if (!f) {   // p > 0: particle 0 starts a tile
      const int64_t t = (int64_t)idx[p] - 1;
      const int32_t c = cost[t];
      if (c > kSplit4 / part) {
        const bool dear = c > kSplit2 / part;
        const double h = fmin(pos4[p].w, pos4[p - 1].w);
        int len = dear ? 32 : 64;
        if (gkeys[p] == gkeys[p - 1] && curve_cell(*gp) > 2.0 * h) {
          const float4 w = tile_box[t].w;
          const float R = (float)(2.0 * pos4[p].w * (1.0 + gp->skin) * gp->bunit), e = 0.25f * R;
          const float most = 1.5f * (float)c * (4.18879f * R * R * R) / (8.f * (w.x + e) * (w.y + e) * (w.z + e));
          len = most * 16.f > (float)ucap ? 8 : (most * 32.f > (float)ucap ? 16 : 32);
        }
        f = ((p - tile_start[t]) & (len - 1)) == 0 || morton_jump(*gp, gkeys, p) > (dear ? 2.0 : 4.0) * h;
        if (f) flag[p] = 1u;
      }
    }
    v += f ? 1u : 0u;
  }
  block_exclusive(v, tot);
  if (threadIdx.x == 0) bsum[blockIdx.x] = tot;
}

// ---- candidate lists ---------------------------------------------------------------------------
// One wave builds the lists of one tile (lane = target).  It descends the boxes: the runs of 64
// tiles near its own box, their tiles, and those tiles' runs of 8 particles, tested against the
// runs of its own tile.  Eight runs that pass form a batch of 64 candidates (lane = candidate),
// which is tested against the 64 targets on the matrix cores:
//   r^2 - (h_a' + h_b')^2 = -2 x_a.x_b - 2 h_a' h_b' + w_a + w_b,  w = |x|^2 - h'^2
// (h' = (1 + skin) h, x relative to the tile's centre).  Each of the four components and w goes in
// as two FP16 parts (hi = f16(v), lo = f16(v - hi)); hi.hi, hi.lo and lo.hi of four components and
// the parts of the two w are 16 products, so one v_mfma_f32_32x32x16_f16 takes a block of 32 x 32
// pairs and four take the batch (128 of the SIMD's cycles; 10 FP64 operations a pair on the vector
// ALUs are 2560).  The sign bits are shifted into one 64-bit mask of hits per target, one v_alignbit
// per 64 pairs.
// The lists only have to contain the exact sets (the density pass takes the exact FP64 decision), so
// each w is lowered by kListBand (|x|^2 + h'^2), more than the test can be off: with M = |x_a|^2 +
// |x_b|^2 + h_a'^2 + h_b'^2 the parts leave out at most 2^-22 of a value, the product lo.lo 2^-22 of
// hi.hi, and the FP32 inputs and the accumulation 40 2^-24 M, in all below 16 2^-22 M against the
// band's 32 2^-22 M (a widening of H by 3e-5).  Lengths are scaled so that the tile's reach is 100.
// A low part below 2^-14 is subnormal in FP16 and may be off by 2^-25 instead: in the ten products and
// w of a pair that adds at most 2^-22 + 2^-25 M, which the other half of the band covers where M >= 1/4.
// A tile with a target of h' < 1/2 (its reach 200 times h' or more) is tested pair by pair.
// In a tile so wide that the band would lengthen its lists (centre-to-corner above 8 of its smallest
// h) every hit is tested again from the FP32 coordinates' differences.  Pair by pair, in FP64, are tested
// a batch with a candidate beyond FP16's range, such tiles, and those of a periodic box less than twice
// their reach across.
// A candidate hit by any target joins the union, as its next member, and each target appends the
// local indices of its hits to its list, ascending.
// Bound by instruction issue (about 490 vector instructions a batch, half of them the appends, and
// their latency: 4 waves a SIMD) and, over the launch, by its dearest tiles.  Measured against a
// cell grid of two smoothing lengths with an FP64 test of every candidate by every lane: 1M-particle
// snapshot 3.34 -> 0.80 ms, 2M-particle star in a run 3.19 -> 1.32 ms (FP64 skin 0.08) and
// 3.44 -> 1.4 ms (skin 0.14), 15k-particle star 0.38 -> 0.145 ms.
struct BuildArgs {
  const double4* __restrict__ pos4;
  const GridInfo* __restrict__ grid;
  const int32_t* __restrict__ tile_start;
  const int32_t* __restrict__ tile_cnt;
  const Box* __restrict__ tile_box;
  const Box* __restrict__ sub_box;
  const Box* __restrict__ super_box;
  const uint32_t* __restrict__ tile_uoff;
  int64_t capw, upool;
  int cap, ucap;
  int32_t* __restrict__ tile_u;
  int32_t* __restrict__ tile_usize;
  uint16_t* __restrict__ nbr16;     // candidate slot lists
  int32_t* __restrict__ count;       // candidates per particle
  int lanes;                         // slots per particle (lanes per target of the pair passes)
  int cap_sl;                        // entries a slot holds
  DevStatus* status;
};

constexpr float kListBand = 0x1p-17f;
constexpr int kRuns = 304;   // near runs collected before they are tested (12.5 KB of LDS: 13 waves a CU)
template <bool PER, int NL>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(4))) void k_build_tiles(BuildArgs B) {
  __shared__ int32_t q_tile[128];        // ring: near tiles waiting for their runs to be tested
  __shared__ int32_t q_run[kRuns];       // near runs: first particle ...
  __shared__ uint8_t q_len[kRuns];       //   ... and length
  __shared__ float4 own_c[8], own_w[8];  // the tile's own runs
  __shared__ float4 cand[64];            // a batch's scaled coordinates, by bit of the masks (wide tiles)
  uint32_t* self = reinterpret_cast<uint32_t*>(cand);   // then its candidate that is the lane's own particle
  __shared__ __align__(16) uint16_t ring[64 * kRingRow];
  const int lane = threadIdx.x;
  const GridInfo& g = *B.grid;
  const double box = g.box, s1 = 1.0 + g.skin;
  const float s1f = (float)s1 * (1.0f + 1e-5f), boxf = (float)(box * g.bunit);
  const double ibu = 1.0 / g.bunit;
  const int64_t ntiles = g.ntiles, ns = (ntiles + 63) / 64;
  const unsigned long long lt = lane ? (~0ull >> (64 - lane)) : 0ull;
  // candidate lane c of a batch is bit cbit of word cword of the masks (the order in which the
  // products' rows come out)
  const int cword = (lane >> 2) & 1, cbit = 16 * (lane >> 5) + 4 * ((lane >> 3) & 3) + (lane & 3);
  for (int64_t k_ = blockIdx.x / SPH_XCD, chunk_ = xcd_chunk(ntiles); k_ < chunk_; k_ += gridDim.x / SPH_XCD) {
    const int64_t t = (int64_t)(blockIdx.x % SPH_XCD) * chunk_ + k_;
    if (t >= ntiles) break;
    const int32_t ts = B.tile_start[t], tcnt = B.tile_cnt[t];
    const bool valid = lane < tcnt;
    const int32_t a = ts + lane;
    const double4 pa = valid ? B.pos4[a] : make_double4(0.0, 0.0, 0.0, 0.0);
    const Box own = B.tile_box[t];
    const int nown = (tcnt + 7) >> 3;
    __syncthreads();
    if (lane < nown) {
      const Box b = B.sub_box[(ts >> 3) + t + lane];
      own_c[lane] = b.c;
      own_w[lane] = b.w;
    }
    __syncthreads();
    const uint32_t uoff = B.tile_uoff[t];
    int ucap = (int)((int64_t)tcnt * B.cap < B.ucap ? (int64_t)tcnt * B.cap : B.ucap);
    if ((int64_t)uoff + ucap > B.upool) {
      ucap = 0;
      if (lane == 0) latch_error(B.status, SPH_E_NGB_CAPACITY, -1);
    }
    int32_t* U = B.tile_u + uoff;
    const double c0 = g.org[0] + own.c.x * ibu, c1 = g.org[1] + own.c.y * ibu, c2 = g.org[2] + own.c.z * ibu;
    const float rt2 = own.w.x * own.w.x + own.w.y * own.w.y + own.w.z * own.w.z;
    const float sc = 100.f / (sqrtf(rt2) + 2.f * own.c.w * s1f + 1e-30f);
    const float reach = (sqrtf(rt2) + own.c.w * s1f) * sc * (1.f + 1e-5f);
    const double scd = sc * g.bunit;   // from the caller's lengths
    // scaled components; a lane without a (finite) particle, or with one out of every target's reach,
    // never hits (w beyond any -h'^2); returns |x|^2 + h'^2, which must stay below kListMax in FP16
    auto lift = [&](const double4& p, bool in, float& x, float& y, float& z, float& h, float& w) -> float {
      x = (float)(min_image(p.x - c0, (int)PER, box) * scd);
      y = (float)(min_image(p.y - c1, (int)PER, box) * scd);
      z = (float)(min_image(p.z - c2, (int)PER, box) * scd);
      h = (float)(p.w * (s1 * scd));
      const float r2 = x * x + y * y + z * z, h2 = h * h, far = reach + h;
      w = (r2 - h2) - kListBand * (r2 + h2);
      if (!(in && r2 < far * far && h2 < 1e30f)) {   // (NaN fails too)
        x = y = z = h = 0.f;
        w = 60000.f;
        return 0.f;
      }
      return r2 + h2;
    };
    constexpr float kListMax = 3e4f;
    f16x8 T[2];
    const float hmn = (float)(wave_min_d(valid ? pa.w : 1e300) * g.bunit);
    const bool wide = rt2 > 64.f * hmn * hmn;
    bool by_pair = false;
    float tx, ty, tz, th;
    {
      float w;
      const float m = lift(pa, valid, tx, ty, tz, th, w);
      lift_operands<true>(tx, ty, tz, th, w, T);
      by_pair = __ballot(m > kListMax || (valid && !(th >= 0.5f))) != 0ull;
    }
    if (PER) by_pair = by_pair || fmaxf(own.w.x, fmaxf(own.w.y, own.w.z)) + (own.c.w + (float)(g.hmax * g.bunit)) * s1f > 0.499f * boxf;
    ListOut<NL> out;
    out.ring = ring + kRingRow * lane;
    out.slot0 = reinterpret_cast<uint4*>(B.nbr16) + (valid ? (int64_t)a : 0) * NL;
    out.gstride = B.capw * NL;
    out.cap_sl = B.cap_sl;
    out.cnt = out.stored = 0;
    int usize = 0;
    // candidate of batch k of nb: its runs are k, k + nb, ... of those collected, lane / 8 the run and
    // lane % 8 the particle.  A batch is thus spread over the whole neighbourhood and a target's hits
    // come evenly from all batches (with neighbouring runs in one batch a target near them hits most
    // of it, and the wave waits for the target with the most hits: 0.94 against 0.80 ms).
    auto fetch = [&](int k, int nb, int nr, double4& pb) -> int32_t {
      const int q = k + nb * (lane >> 3), r = lane & 7;
      const bool in = k < nb && q < nr && r < (int)q_len[q < kRuns ? q : 0];
      const int32_t b = in ? q_run[q] + r : -1;
      pb = in ? B.pos4[b] : make_double4(0.0, 0.0, 0.0, 0.0);
      return b;
    };
    auto batch = [&](int32_t b, const double4& pb) {
      const bool in = b >= 0;
      uint32_t m0, m1;
      float x, y, z, h, w;
      const float mag = lift(pb, in, x, y, z, h, w);
      if (!by_pair && !__ballot(mag > kListMax)) {
        f16x8 C[2];
        lift_operands<false>(x, y, z, h, w, C);
        uint32_t q[2];
#pragma unroll
        for (int tb = 0; tb < 2; ++tb) {
          const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
          const f32x16 D0 = __builtin_amdgcn_mfma_f32_32x32x16_f16(C[0], T[tb], zero, 0, 0, 0);
          const f32x16 D1 = __builtin_amdgcn_mfma_f32_32x32x16_f16(C[1], T[tb], zero, 0, 0, 0);
          uint32_t q0 = 0u, q1 = 0u;
#pragma unroll
          for (int e = 15; e >= 0; --e) {
            q0 = __builtin_amdgcn_alignbit(q0, __float_as_uint(D0[e]), 31u);
            q1 = __builtin_amdgcn_alignbit(q1, __float_as_uint(D1[e]), 31u);
          }
          q[tb] = q0 | (q1 << 16);
        }
        // lane l < 32 holds rows 8 i + j (upper lanes: 8 i + 4 + j) of targets l and 32 + l: each
        // lane receives both halves of its own target
        m0 = q[0];
        m1 = q[1];
        swap32(m0, m1);
        if (wide && __ballot((m0 | m1) != 0u)) {
          __syncthreads();
          cand[32 * cword + cbit] = make_float4(x, y, z, h);
          __syncthreads();
          // coordinates rounded to FP32 (their differences to 2^-22 |x|, |x| < 2 sqrt(kListMax)): the
          // support widened by 1e-5 and 2e-4 of the scaled unit holds every pair of the exact test
          auto again = [&](uint32_t m, int word) -> uint32_t {
            uint32_t keep = 0u;
            while (m) {
              const int b = __builtin_ctz(m);
              m &= m - 1;
              const float4 c = cand[32 * word + b];
              const float dx = tx - c.x, dy = ty - c.y, dz = tz - c.z, H = (th + c.w) * (1.f + 1e-5f) + 2e-4f;
              keep |= (dx * dx + dy * dy + dz * dz < H * H ? 1u : 0u) << b;
            }
            return keep;
          };
          m0 = again(m0, 0);
          m1 = again(m1, 1);
        }
      } else {
        m0 = m1 = 0u;
        for (int j = 0; j < 64; ++j) {
          const double4 q = make_double4(__shfl(in ? pb.x : __builtin_nan(""), j, 64), __shfl(pb.y, j, 64),
                                         __shfl(pb.z, j, 64), __shfl(pb.w, j, 64));
          const double dx = min_image(pa.x - q.x, (int)PER, box), dy = min_image(pa.y - q.y, (int)PER, box),
                       dz = min_image(pa.z - q.z, (int)PER, box);
          const double H = (pa.w + q.w) * s1 * (1.0 + 0x1p-40);
          const uint32_t bit = (valid && dx * dx + dy * dy + dz * dz < H * H ? 1u : 0u)
                               << (16 * (j >> 5) + 4 * ((j >> 3) & 3) + (j & 3));
          if ((j >> 2) & 1) m1 |= bit;
          else m0 |= bit;
        }
      }
      // a particle is not its own neighbour
      const int ta = b - ts;   // the target this candidate is, if it is of the tile
      if (__ballot(in && ta >= 0 && ta < tcnt)) {
        __syncthreads();
        self[lane] = 64u;
        __syncthreads();
        if (in && ta >= 0 && ta < tcnt) self[ta] = (uint32_t)(32 * cword + cbit);
        __syncthreads();
        const uint32_t sb = self[lane];
        if (sb < 32u) m0 &= ~(1u << sb);
        else if (sb < 64u) m1 &= ~(1u << (sb - 32u));
      }
      const uint32_t u0 = wave_or(m0), u1 = wave_or(m1);   // the batch's union members
      if (!(u0 | u1)) return;
      const int n0 = __builtin_popcount(u0);
      {
        const uint32_t uw = cword ? u1 : u0;
        const int loc = usize + (cword ? n0 : 0) + __builtin_popcount(uw & ((1u << cbit) - 1u));
        if (((uw >> cbit) & 1u) && loc < ucap) U[loc] = b;
      }
      const int last = ucap > 0 ? ucap - 1 : 0;
      out.append(m0, m1, u0, u1, usize, last);
      usize += n0 + __builtin_popcount(u1);
    };
    int nt = 0, ht = 0, nr = 0;      // tiles waiting (and the ring's head), runs collected (wave-uniform)
    int64_t s0 = -64;                // first of the current 64 runs of 64 tiles, and those near
    unsigned long long sm = 0ull;
    bool more = true;
    for (;;) {
      if (nr > kRuns - 64 || (!more && nt == 0 && nr > 0)) {   // the batches of the collected runs
        const int nb = (nr + 7) >> 3;
        __syncthreads();
        double4 p0;
        int32_t b0 = fetch(0, nb, nr, p0);
#pragma unroll 1
        for (int k = 0; k < nb; ++k) {   // the next batch's loads are in flight
          double4 p1;
          const int32_t b1 = fetch(k + 1, nb, nr, p1);
          batch(b0, p0);
          p0 = p1;
          b0 = b1;
        }
        nr = 0;
        __syncthreads();
        continue;
      }
      if (nt >= 8 || (!more && nt > 0)) {   // the runs of 8 tiles, against the tile's own runs
        const int k = nt < 8 ? nt : 8;
        const int gi = lane >> 3, r = lane & 7;
        bool near = false;
        int32_t first = 0, len = 0;
        if (gi < k) {
          const int32_t u = q_tile[(ht + gi) & 127];
          first = B.tile_start[u] + 8 * r;
          len = B.tile_cnt[u] - 8 * r;
          len = len < 8 ? len : 8;
          if (len > 0) {
            const Box b = B.sub_box[((first - 8 * r) >> 3) + u + r];
            for (int o = 0; o < nown; ++o) near = near || boxes_near<PER>(own_c[o], own_w[o], b.c, b.w, s1f, boxf);
          }
        }
        const unsigned long long m = __ballot(near);
        if (near) {
          const int k2 = nr + __popcll(m & lt);
          q_run[k2] = first;
          q_len[k2] = (uint8_t)len;
        }
        nr += __popcll(m);
        nt -= k;
        ht += k;
        __syncthreads();
        continue;
      }
      if (sm) {   // the tiles of the next near run of 64
        const int64_t u = (s0 + __builtin_ctzll(sm)) * 64 + lane;
        sm &= sm - 1;
        bool near = false;
        if (u < ntiles) {
          const Box b = B.tile_box[u];
          near = boxes_near<PER>(own.c, own.w, b.c, b.w, s1f, boxf);
        }
        const unsigned long long m = __ballot(near);
        if (near) q_tile[(ht + nt + __popcll(m & lt)) & 127] = (int32_t)u;
        nt += __popcll(m);
        __syncthreads();
        continue;
      }
      if (!more) break;
      s0 += 64;
      if (s0 >= ns) {
        more = false;
        continue;
      }
      bool near = false;
      if (s0 + lane < ns) {
        const Box b = B.super_box[s0 + lane];
        near = boxes_near<PER>(own.c, own.w, b.c, b.w, s1f, boxf);
      }
      sm = __ballot(near);
    }
    if (valid) out.finish();
    if (valid) B.count[a] = out.cnt < B.cap ? out.cnt : B.cap;
    if (lane == 0) B.tile_usize[t] = usize < ucap ? usize : ucap;
    if (usize > ucap || out.cnt > B.cap) latch_error(B.status, SPH_E_NGB_CAPACITY, valid ? a : -1);
  }
}

__global__ __launch_bounds__(kB) void k_count_stats(const int32_t* __restrict__ cnt, int64_t n,
                                                    unsigned long long* total, int32_t* mx) {
  unsigned long long s = 0;
  int m = 0;
  for (int64_t a = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; a < n; a += (int64_t)gridDim.x * blockDim.x) {
    s += (unsigned long long)cnt[a];
    m = cnt[a] > m ? cnt[a] : m;
  }
  for (int off = 32; off > 0; off >>= 1) {
    s += __shfl_xor(s, off, 64);
    int o = __shfl_xor(m, off, 64);
    m = o > m ? o : m;
  }
  if ((threadIdx.x & 63) == 0) {
    atomicAdd(total, s);
    atomicMax(mx, m);
  }
}

// Permutes the state arrays in place along c->vals, as many at a time as the staging area holds: the
// candidate-list buffer (at least 80 bytes a particle), whose lists the build that follows rewrites.  type
// comes last: the crust arrays are gathered with its old order.
struct PermArray {
  void* p;
  int elem;
  bool crust;
  void* to;   // gathered there for good (a second buffer), or nullptr: back into p
};
static sph_status permute_arrays(sph_ctx* c, const PermArray* A, int m, const int8_t* type, int64_t n) {
  char* stage = reinterpret_cast<char*>(c->nbr16s);
  const size_t room = (size_t)c->capw * (size_t)(c->cap_s + 32) * sizeof(uint16_t);
  const unsigned nb = grid_for(n, kB);
  for (int k = 0; k < m;) {
    PermBatch B{};
    B.type = type;
    size_t used = 0;
    while (k < m && B.na < kPermMax) {
      const size_t bytes = A[k].to ? 0 : ((size_t)n * A[k].elem + 255) & ~(size_t)255;
      if (B.na > 0 && used + bytes > room) break;
      B.arr[B.na] = A[k].p;
      B.stage[B.na] = A[k].to ? (char*)A[k].to : stage + used;
      B.back[B.na] = A[k].to ? 0 : 1;
      B.elem[B.na] = (uint8_t)A[k].elem;
      B.crust[B.na] = A[k].crust ? 1 : 0;
      used += bytes;
      ++B.na;
      ++k;
    }
    hipLaunchKernelGGL(k_permute_gather, dim3(nb), dim3(kB), 0, c->stream, B, c->vals, n);
    hipLaunchKernelGGL(k_permute_copy, dim3(nb), dim3(kB), 0, c->stream, B, n);
  }
  HIP_TRY(hipGetLastError());
  return SPH_OK;
}

}  // namespace

// The union pool is sized to what the tiles reserve: read the reservation total and grow the
// pool (by a quarter more than needed) when it does not fit.  Waits for the stream.
static sph_status ensure_pool(sph_ctx* c) {
  // ntiles, upool_used and nstress are adjacent in GridInfo: one copy brings all three
  static_assert(offsetof(GridInfo, upool_used) == offsetof(GridInfo, ntiles) + 4 &&
                    offsetof(GridInfo, nstress) == offsetof(GridInfo, ntiles) + 8,
                "GridInfo layout");
  HIP_TRY(hipMemcpyAsync(c->drift_host, &c->grid->ntiles, 3 * sizeof(uint32_t), hipMemcpyDeviceToHost, c->stream));
  HIP_TRY(hipStreamSynchronize(c->stream));
  const uint32_t used = c->drift_host[1];
  c->ntiles = c->drift_host[0];
  c->nstress = c->drift_host[2];
  c->stress_heavy = 2ull * c->drift_host[2] > (unsigned long long)c->drift_host[0];
  if ((int64_t)used <= c->upool) return SPH_OK;
  int64_t want = (int64_t)used + (int64_t)used / 4;
  if (want > (int64_t)0xffffffffll) want = (int64_t)0xffffffffll;
  HIP_TRY(hipFree(c->tile_u));
  c->tile_u = nullptr;
  c->upool = 0;
  if (hipMalloc((void**)&c->tile_u, sizeof(int32_t) * (size_t)want) != hipSuccess) {
    c->tile_u = nullptr;
    return SPH_E_OOM;
  }
  c->upool = want;
  ++c->graph_epoch;   // captured kernels hold the old pool pointer
  return SPH_OK;
}

static unsigned tile_grid(int64_t cap_tiles) {
  return (unsigned)(cap_tiles < 65536 ? cap_tiles : 65536);
}
// A multiple of the XCD count.  An empty workgroup of the pair passes costs 0.2 ns of dispatch each:
// 14 us a pass when a grid of 65536 is launched for no tile.
unsigned tile_launch(const sph_ctx* c) {
  const unsigned all = tile_grid(c->cap_tiles);
  if (c->p.graph) return all;
  const unsigned t = (c->ntiles + SPH_XCD - 1) / SPH_XCD * SPH_XCD;
  return t < 1 ? SPH_XCD : (t < all ? t : all);
}

template <bool PER>
static void launch_build_per(const BuildArgs& B, dim3 grid, hipStream_t s) {
  if (B.lanes == 1)
    hipLaunchKernelGGL(HIP_KERNEL_NAME(k_build_tiles<PER, 1>), grid, dim3(64), 0, s, B);
  else if (B.lanes == 2)
    hipLaunchKernelGGL(HIP_KERNEL_NAME(k_build_tiles<PER, 2>), grid, dim3(64), 0, s, B);
  else
    hipLaunchKernelGGL(HIP_KERNEL_NAME(k_build_tiles<PER, 4>), grid, dim3(64), 0, s, B);
}
static void launch_build(const BuildArgs& B, bool per, dim3 grid, hipStream_t s) {
  if (per) launch_build_per<true>(B, grid, s);
  else launch_build_per<false>(B, grid, s);
}

// Candidate-list build: every particle array of the state is reordered along the global Morton curve (the
// outputs only when outputs_recomputed is false, the half-step copies only when it is true), tiles are cut
// from that order and each tile's candidates are collected, through the boxes of runs of particles or, where
// the sums keep their order, in very large sets and with a wide skin, through the multi-level grid; the positions and h at the list build are kept
// for the drift test.
sph_status sph_rebin(sph_ctx* c, sph_state* st, bool outputs_recomputed) {
  const int64_t n = st->n;
  hipStream_t s = c->stream;
  const unsigned nb = grid_for(n, kB), nb4 = grid_for(n, 1024);
  unsigned nred = nb < 1024 ? nb : 1024;
  sph_status e;
  const bool cells = keeps_sum_order(c->p) || wide_skin(c->p, n) || n > kBoxesMost;
  c->tile_len = !cells && small_tiles(c->p, n) ? 32 : 64;
  hipLaunchKernelGGL(k_bounds, dim3(nred), dim3(kB), 0, s, st->x, st->y, st->z, st->h, n, c->sort.partial);
  hipLaunchKernelGGL(k_grid_setup1, dim3(1), dim3(64), 0, s, c->grid, c->sort.partial, (int)nred, c->p.periodic,
                     c->p.box, c->p.skin, c->status);
  hipLaunchKernelGGL(k_gkeys, dim3(nb), dim3(kB), 0, s, st->x, st->y, st->z, n, c->grid, c->keys, c->vals);
  if ((e = sph_sort_pairs(c, c->keys, c->vals, n))) return e;
  {
    const bool in_place = c->p.graph || exact_lists_written(c);
    PermArray A[64];
    int m = 0;
    for (double* a : {st->x, st->y, st->z, st->vx, st->vy, st->vz, st->u, st->h}) A[m++] = {a, 8, false, nullptr};
    for (int k = 0; k < 6; ++k) A[m++] = {st->S + k * n, 8, true, nullptr};
    if (!outputs_recomputed) {
      for (double* a : {st->D, st->rho, st->P, st->cs, st->ax, st->ay, st->az, st->dudt}) A[m++] = {a, 8, false, nullptr};
      for (int k = 0; k < 6; ++k) A[m++] = {st->dSdt + k * n, 8, true, nullptr};
    } else {   // state that the next evaluation reads although it is an output
      if (c->p.density_mode == SPH_DENS_CONTINUITY) A[m++] = {st->D, 8, false, nullptr};
      if (c->p.dtP_mode == SPH_DTP_LAGGED) A[m++] = {st->P, 8, false, nullptr};
      // the step's half-step copies, into their second buffer (outside a step nothing reads them); in
      // place where captured kicks hold the first one (a new capture costs more than the copy) or exact
      // lists take the second one's room
      for (int k = 0; k < SPH_HALF_FIELDS; ++k)
        if (k < 10 || c->p.density_mode == SPH_DENS_CONTINUITY)
          A[m++] = {c->half + (int64_t)k * c->capacity, 8, k >= 4 && k < 10,
                    in_place ? nullptr : c->half_alt + (int64_t)k * c->capacity};
    }
    A[m++] = {st->id, 4, false, nullptr};
    if (st->star) A[m++] = {st->star, 4, false, nullptr};
    A[m++] = {st->broken, 1, false, nullptr};
    A[m++] = {st->type, 1, false, nullptr};
    if ((e = permute_arrays(c, A, m, st->type, n))) return e;
    if (outputs_recomputed && !in_place) {
      double* t = c->half;
      c->half = c->half_alt;
      c->half_alt = t;
      ++c->graph_epoch;   // a graph captured before would hold the old buffer
    }
    hipLaunchKernelGGL(k_pack_pos, dim3(nb), dim3(kB), 0, s, st->x, st->y, st->z, st->h, st->star, c->stars, n, c->pos4,
                       c->p.precision == SPH_FP32 ? c->pos4f : nullptr, c->pos_build, st->type, st->dSdt, c->sdot);
  }
  // tile table: Morton cuts, then tiles with many particles near them are split
  uint32_t* flag = reinterpret_cast<uint32_t*>(c->tmp);
  uint32_t* idx = flag + c->capw;
  uint32_t* bsum = c->sort.scan_bsum;
  hipLaunchKernelGGL(k_tile_flags, dim3(nb4), dim3(kB), 0, s, c->keys, st->h, n, c->grid, tile_cut_of(c->p), c->tile_len, flag, bsum);
  const bool per = c->p.periodic != 0;
  const dim3 tgrid(tile_grid(c->cap_tiles));
  auto starts = [&] {
    sph_scan_rows(c, bsum, (int)nb4, &c->grid->ntiles);
    hipLaunchKernelGGL(k_tile_starts, dim3(nb4), dim3(kB), 0, s, flag, bsum, n, idx, c->tile_start);
  };
  uint32_t* crust = c->tile_st;   // until the build marks the tiles' unions there
  if (cells) {
    starts();
    hipLaunchKernelGGL(k_tile_len, dim3(tgrid.x < 1024 ? tgrid.x : 1024), dim3(kB), 0, s, c->grid, n, c->tile_start,
                       c->tile_cnt);
    if ((e = grid_prepare(c, n)) || (e = grid_split_tiles(c, n, flag, idx, tgrid.x, bsum))) return e;
    starts();
    hipLaunchKernelGGL(k_tile_crust, dim3(tgrid.x < 16384 ? tgrid.x : 16384), dim3(256), 0, s, c->grid, n, c->tile_start,
                       st->type, c->tile_cnt, crust);
  } else {
    auto boxes = [&] {
      hipLaunchKernelGGL(k_tile_boxes, tgrid, dim3(64), 0, s, c->grid, c->pos4, n, c->tile_start, st->type, c->tile_cnt,
                         crust, c->tile_box, c->sub_box);
      hipLaunchKernelGGL(k_super_boxes, dim3((tgrid.x + 63) / 64), dim3(64), 0, s, c->grid, c->tile_box, c->super_box);
    };
    starts();
    boxes();
    if (per)
      hipLaunchKernelGGL(HIP_KERNEL_NAME(k_tile_cost<true>), tgrid, dim3(64), 0, s, c->grid, c->tile_cnt, c->tile_box,
                         c->super_box, c->tile_usize);
    else
      hipLaunchKernelGGL(HIP_KERNEL_NAME(k_tile_cost<false>), tgrid, dim3(64), 0, s, c->grid, c->tile_cnt, c->tile_box,
                         c->super_box, c->tile_usize);
    hipLaunchKernelGGL(k_tile_split, dim3(nb4), dim3(kB), 0, s, flag, idx, n, c->tile_start, c->tile_usize,
                       c->keys, c->pos4, c->tile_box, c->ucap, c->grid, bsum);
    starts();
    boxes();
  }
  // reservations in the union pool and the stress pass's work list; sizes read back with them
  hipLaunchKernelGGL(k_tile_sums, dim3(nb4), dim3(kB), 0, s, c->grid, c->tile_cnt, crust, c->cap_s, c->ucap, bsum, (int)nb4);
  sph_scan_rows(c, bsum, (int)nb4, &c->grid->upool_used, 2);
  hipLaunchKernelGGL(k_tile_offsets, dim3(nb4), dim3(kB), 0, s, c->grid, c->tile_cnt, crust, c->cap_s, c->ucap, bsum,
                     (int)nb4, c->tile_uoff, c->stress_tiles);
  HIP_TRY(hipGetLastError());
  if ((e = ensure_pool(c))) return e;   // also brings the number of tiles
  if (cells) {
    if ((e = grid_build_lists(c, n, tile_launch(c)))) return e;
  } else {
    BuildArgs B;
    B.pos4 = c->pos4; B.grid = c->grid; B.tile_box = c->tile_box; B.sub_box = c->sub_box; B.super_box = c->super_box;
    B.capw = c->capw; B.cap = c->cap_s; B.ucap = c->ucap;
    B.lanes = pass_lanes(c->p); B.cap_sl = cand_slot_capacity(c->cap_s, B.lanes);
    B.tile_start = c->tile_start; B.tile_cnt = c->tile_cnt; B.tile_uoff = c->tile_uoff; B.upool = c->upool;
    B.tile_u = c->tile_u; B.tile_usize = c->tile_usize; B.nbr16 = c->nbr16s; B.count = c->nbr_count_s;
    B.status = c->status;
    launch_build(B, per, dim3(tile_launch(c)), s);
  }
  hipLaunchKernelGGL(k_tile_union_type, dim3(tile_launch(c)), dim3(64), 0, s, c->grid, c->tile_start,
                     c->tile_cnt, c->tile_uoff, c->tile_usize, c->tile_u, st->type, c->tile_st);
  HIP_TRY(hipGetLastError());
  return SPH_OK;
}

// Skin test of the current positions and h against the last build (for sph_build_cells; inside
// sph_step the test is fused into the drift kernel).
__global__ __launch_bounds__(kB) void k_drift_check(const double* __restrict__ x, const double* __restrict__ y,
                                                    const double* __restrict__ z, const double* __restrict__ h,
                                                    const double4* __restrict__ pb, int64_t n,
                                                    const GridInfo* __restrict__ gp, uint32_t id,
                                                    uint32_t* __restrict__ flag) {
  const int64_t a = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  bool out = false;
  if (a < n) {
    const GridInfo& g = *gp;
    const double4 b = pb[a];
    out = skin_exceeded(min_image(x[a] - b.x, g.periodic, g.box), min_image(y[a] - b.y, g.periodic, g.box),
                        min_image(z[a] - b.z, g.periodic, g.box), h[a], b, g.skin);
  }
  // one plain store a workgroup, all of the same value: after a new snapshot every particle is out, and
  // an atomic for each took 183 us at 1M particles
  if (__syncthreads_or(out) && threadIdx.x == 0) *flag = id;
}

sph_status launch_drift_check(sph_ctx* c, sph_state* st) {
  hipLaunchKernelGGL(k_drift_check, dim3(grid_for(st->n, kB)), dim3(kB), 0, c->stream, st->x, st->y, st->z,
                     st->h, c->pos_build, st->n, c->grid, c->check_id, c->drift_flag);
  HIP_TRY(hipGetLastError());
  return SPH_OK;
}

// Pack the position records the pair passes read, in the current particle order.
sph_status launch_pack(sph_ctx* c, sph_state* st) {
  const int64_t n = st->n;
  hipLaunchKernelGGL(k_pack_pos, dim3(grid_for(n, kB)), dim3(kB), 0, c->stream, st->x, st->y, st->z, st->h,
                     st->star, c->stars, n, c->pos4, c->p.precision == SPH_FP32 ? c->pos4f : nullptr, nullptr, nullptr, nullptr,
                     nullptr);
  HIP_TRY(hipGetLastError());
  return SPH_OK;
}

__global__ __launch_bounds__(kB) void k_union_stats(const int32_t* __restrict__ usize, const GridInfo* __restrict__ gp,
                                                    unsigned long long* total) {
  unsigned long long s = 0;
  const int64_t nt = gp->ntiles;
  for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < nt; t += (int64_t)gridDim.x * blockDim.x)
    s += (unsigned long long)usize[t];
  for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
  if ((threadIdx.x & 63) == 0) atomicAdd(total, s);
}

sph_status sph_count_stats(sph_ctx* c, sph_list_stats* out) {
  struct R { unsigned long long t, u, cs; int32_t m, ms; };
  R* d = nullptr;
  if (hipMalloc((void**)&d, sizeof(R)) != hipSuccess) return SPH_E_OOM;
  R h = {0ull, 0ull, 0ull, 0, 0};
  sph_status e = SPH_OK;
  if (hipMemcpy(d, &h, sizeof(R), hipMemcpyHostToDevice) != hipSuccess) e = SPH_E_HIP;
  if (!e && c->n > 0 && c->lists_valid) {
    unsigned nb = grid_for(c->n, kB);
    nb = nb < 1024 ? nb : 1024;
    if (c->gen >= 2)
      hipLaunchKernelGGL(k_count_stats, dim3(nb), dim3(kB), 0, c->stream, c->nbr_count, c->n, &d->t, &d->m);
    hipLaunchKernelGGL(k_count_stats, dim3(nb), dim3(kB), 0, c->stream, c->nbr_count_s, c->n, &d->cs, &d->ms);
    hipLaunchKernelGGL(k_union_stats, dim3(256), dim3(kB), 0, c->stream, c->tile_usize, c->grid, &d->u);
    if (hipStreamSynchronize(c->stream) != hipSuccess) e = SPH_E_HIP;
  }
  if (!e && hipMemcpy(&h, d, sizeof(R), hipMemcpyDeviceToHost) != hipSuccess) e = SPH_E_HIP;
  (void)hipFree(d);
  out->pairs = (int64_t)h.t;
  out->max_count = h.m;
  out->pad = 0;
  out->union_total = (int64_t)h.u;
  out->candidates = (int64_t)h.cs;
  out->rebuilds = c->rebuilds;
  out->tiles = 0;
  if (!e && c->n > 0 && c->lists_valid) {
    GridInfo g;
    if (hipMemcpy(&g, c->grid, sizeof(g), hipMemcpyDeviceToHost) != hipSuccess) return SPH_E_HIP;
    out->tiles = (int64_t)g.ntiles;
  }
  return e;
}

// ---- list statistics without device allocation ------------------------------------------------
// Counters of sph_neighbour_stats_noalloc: exact pairs, union members, candidates (64-bit) and
// the longest exact and candidate lists (32-bit, in the fourth and fifth words).  One copy per
// GPU, held until the process ends; every call on a GPU uses that GPU's copy.  Host code never
// names the array in a kernel argument or copy: it uses the device address looked up once per
// device by stats_scratch_init.
constexpr int kStatWords = 8;
static __device__ __align__(256) unsigned long long scratch[kStatWords];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
unsigned long long* g_scratch_addr[kMaxDevices] = {};

__global__ void k_clear_words(unsigned long long* __restrict__ w, int n) {
  if ((int)threadIdx.x < n) w[threadIdx.x] = 0ull;
}
}  // namespace

sph_status stats_scratch_init(sph_ctx* c) {
  if (c->device < 0 || c->device >= kMaxDevices) return SPH_E_ARG;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_addr[c->device]) {
    int cur = -1;
    HIP_TRY(hipGetDevice(&cur));
    if (cur != c->device) HIP_TRY(hipSetDevice(c->device));
    void* ptr = nullptr;
    const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (cur != c->device) (void)hipSetDevice(cur);
    if (e != hipSuccess || !ptr) return SPH_E_HIP;
    g_scratch_addr[c->device] = (unsigned long long*)ptr;
  }
  c->stats_scratch = g_scratch_addr[c->device];
  return SPH_OK;
}

extern "C" sph_status sph_neighbour_stats_noalloc(sph_ctx* c, sph_list_stats* out) {
  if (!c) return note(nullptr, SPH_E_ARG, "context is NULL");
  if (!out) return note(c, SPH_E_ARG, "out is NULL");
  unsigned long long* d = c->stats_scratch;
  if (!d) return note(c, SPH_E_HIP, "no statistics scratch address for device %d", c->device);
  hipLaunchKernelGGL(k_clear_words, dim3(1), dim3(64), 0, c->stream, d, kStatWords);
  int32_t* mx = reinterpret_cast<int32_t*>(d + 3);   // words 3 and 4 hold the two maxima
  if (c->n > 0 && c->lists_valid) {
    unsigned nb = grid_for(c->n, kB);
    nb = nb < 1024 ? nb : 1024;
    if (c->gen >= 2) hipLaunchKernelGGL(k_count_stats, dim3(nb), dim3(kB), 0, c->stream, c->nbr_count, c->n, d, mx);
    hipLaunchKernelGGL(k_count_stats, dim3(nb), dim3(kB), 0, c->stream, c->nbr_count_s, c->n, d + 2, mx + 2);
    hipLaunchKernelGGL(k_union_stats, dim3(256), dim3(kB), 0, c->stream, c->tile_usize, c->grid, d + 1);
  }
  hipError_t he = hipGetLastError();
  unsigned long long h[kStatWords];
  GridInfo g;
  if (he == hipSuccess) he = hipMemcpyAsync(h, d, sizeof(h), hipMemcpyDeviceToHost, c->stream);
  if (he == hipSuccess && c->n > 0 && c->lists_valid)
    he = hipMemcpyAsync(&g, c->grid, sizeof(g), hipMemcpyDeviceToHost, c->stream);
  if (he == hipSuccess) he = hipStreamSynchronize(c->stream);
  if (he != hipSuccess) return note(c, SPH_E_HIP, "statistics: %s", hipGetErrorString(he));
  int32_t m[4];
  memcpy(m, h + 3, sizeof(m));
  out->pairs = (int64_t)h[0];
  out->union_total = (int64_t)h[1];
  out->candidates = (int64_t)h[2];
  out->max_count = m[0];
  out->pad = 0;
  out->rebuilds = c->rebuilds;
  out->tiles = (c->n > 0 && c->lists_valid) ? (int64_t)g.ntiles : 0;
  return SPH_OK;
}
