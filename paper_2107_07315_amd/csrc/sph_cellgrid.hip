// Candidate-list build on a multi-level cell grid, for FP32 pair sums, for shells in both precisions, for
// FP64 runs with a wide skin (wide_skin) and for very large FP64 sets (kBoxesMost in sph_cells.hip).
//
// Particles are binned into up to four levels by h (factor 2 per level), each with its own uniform
// grid (cell size 2 hmax_l / cell_div) addressed by Morton codes.  A tile searches every level l
// within h_a + hmax_l and skips cells whose box lies farther away.
// Why FP32 runs keep this build while FP64 runs take the box search of sph_cells.hip: the order of
// a tile's union decides which of a target's lanes adds which term, and when, and an FP32 sum's
// rounding with it.  In a star near equilibrium the accelerations are small differences of large
// pair terms, and a rounding difference moves a few particles to the next FP32 position in the steps
// that follow: taken from the other build's order, ten steps of the 2M-particle star differ by
// 2.5e-5 in the accelerations (both orders are equally far from the FP64 values), a perfect lattice
// by 2e-3.  With this build FP32 runs reproduce earlier results bit for bit.
// A shell between an inner and an outer wall keeps it in FP64 too, with tiles of 64 particles and one
// lane to a slot list at every size, so that its sums keep their order: where all particles lie in one
// layer, the radii in a slab differ by 4e-5 of themselves, and the linear fit of sph_diagnostics solves
// normal equations of a condition up to 1e11.  Sums in the other build's order change the state after
// ten steps by 1e-12 at most, and the fit with it by 4e-10 to 1.5e-7 (20k to 290k particles).  Ten steps
// with the record, us, with the other build and with this one: 21k particles 1240 and 1510, 81k 2185 and
// 2580, 290k 4340 and 4790.
#include "sph_build.h"
#include "sph_internal.h"

namespace {

constexpr int kB = 256;

__device__ __forceinline__ int particle_level(double h, const GridInfo& g) {
  double ratio = h / g.hmin;
  int l = 0;
  while (l < g.nlev - 1 && ratio >= (double)(2 << l)) ++l;
  return l;
}

// Per level: largest h and the bounding box of the level's particles (a tile's search at a level
// is clipped to that box, which keeps large-h tiles from enumerating the empty fine cells of
// levels that only occupy the core).
// Each thread keeps the extremes of its particles per level in registers, a wave combines them by
// shuffles and one lane a block and level adds them to the grid with atomics (an LDS atomic for each
// particle's seven values took 57 us at 1M particles).
__global__ __launch_bounds__(kB) void k_level_hmax(const double4* __restrict__ pos4, int64_t n, GridInfo* g) {
  __shared__ unsigned long long red[kB / 64][SPH_MAX_LEV][7];
  const GridInfo& G = *g;
  const int nlev = G.nlev;
  unsigned long long m[SPH_MAX_LEV][7];   // max h bits, low corner, high corner (encoded)
#pragma unroll
  for (int l = 0; l < SPH_MAX_LEV; ++l)
#pragma unroll
    for (int k = 0; k < 7; ++k) m[l][k] = k >= 1 && k < 4 ? ~0ull : 0ull;
  for (int64_t a = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; a < n; a += (int64_t)gridDim.x * blockDim.x) {
    const double4 q = pos4[a];
    const int lev = particle_level(q.w, G);
    const unsigned long long hb = (unsigned long long)__double_as_longlong(q.w);
    const unsigned long long e[3] = {enc_double(q.x), enc_double(q.y), enc_double(q.z)};
#pragma unroll
    for (int l = 0; l < SPH_MAX_LEV; ++l) {
      if (l != lev) continue;
      m[l][0] = hb > m[l][0] ? hb : m[l][0];
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        m[l][1 + d] = e[d] < m[l][1 + d] ? e[d] : m[l][1 + d];
        m[l][4 + d] = e[d] > m[l][4 + d] ? e[d] : m[l][4 + d];
      }
    }
  }
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int l = 0; l < SPH_MAX_LEV; ++l) {
    if (l >= nlev) break;
#pragma unroll
    for (int k = 0; k < 7; ++k) {
      unsigned long long v = m[l][k];
      const bool lo = k >= 1 && k < 4;
      for (int off = 32; off > 0; off >>= 1) {
        const unsigned long long o = __shfl_xor(v, off, 64);
        v = lo ? (o < v ? o : v) : (o > v ? o : v);
      }
      if (lane == 0) red[wave][l][k] = v;
    }
  }
  __syncthreads();
  if ((int)threadIdx.x >= nlev * 7) return;
  const int l = threadIdx.x / 7, k = threadIdx.x % 7;
  const bool lo = k >= 1 && k < 4;
  unsigned long long v = red[0][l][k];
  for (int w = 1; w < kB / 64; ++w) {
    const unsigned long long o = red[w][l][k];
    v = lo ? (o < v ? o : v) : (o > v ? o : v);
  }
  if (k == 0) {
    if (v) atomicMax(&g->hlev_bits[l], v);
  } else if (lo) {
    if (v != ~0ull) atomicMin(&g->lev_lo[l][k - 1], v);
  } else if (v) {
    atomicMax(&g->lev_hi[l][k - 4], v);
  }
}

__global__ void k_grid_setup2(GridInfo* g, int cell_div, int64_t max_cells, DevStatus* st) {
  double hi[3];
  for (int d = 0; d < 3; ++d) hi[d] = g->periodic ? g->box : dec_double(g->enc_hi[d]);
  double grow = 1.0;
  for (int attempt = 0; attempt < 64 && g->hmin > 0.0; ++attempt) {
    uint64_t total = 0;
    bool ok = true;
    for (int l = 0; l < g->nlev; ++l) {
      double hl = __longlong_as_double((long long)g->hlev_bits[l]);
      if (!(hl > 0.0)) hl = g->hmin * (double)(1 << l);
      g->hlev[l] = hl;
      double c = 2.0 * hl / (double)cell_div * grow;
      int bmax = 0;
      for (int d = 0; d < 3; ++d) {
        // counted in FP64: a wide set has more cells than an int counts
        const double cells = g->periodic ? floor(g->box / c) : floor((hi[d] - g->lo[d]) / c) + 1.0;
        if (cells > 1024.0) ok = false;
        const int dim = ok && cells > 1.0 ? (int)cells : 1;
        g->dims[l][d] = dim;
        int b = 0;
        while ((1 << b) < dim) ++b;
        bmax = b > bmax ? b : bmax;
      }
      g->cell[l] = g->periodic ? 0.0 : c;   // periodic: per-dimension sizes below
      g->bits[l] = bmax;
      g->base[l] = (uint32_t)total;
      total += 1ull << (3 * bmax);
    }
    if (ok && total <= (uint64_t)max_cells) {
      g->base[g->nlev] = (uint32_t)total;
      if (g->periodic)
        for (int l = 0; l < g->nlev; ++l) g->cell[l] = g->box / (double)g->dims[l][0];
      return;
    }
    grow *= 1.25;
  }
  // No grid fits: fall back to a single cell (every key 0, memory-safe) and report the error.
  latch_error(st, SPH_E_ARG, -1);
  g->nlev = 1;
  g->cell[0] = 1e300;
  g->dims[0][0] = g->dims[0][1] = g->dims[0][2] = 1;
  g->bits[0] = 0;
  g->base[0] = 0;
  g->base[1] = 1;
}

__device__ __forceinline__ int cell_coord(double x, double lo, double c, int dim) {
  int k = (int)floor((x - lo) / c);
  return k < 0 ? 0 : (k > dim - 1 ? dim - 1 : k);
}

__global__ __launch_bounds__(kB) void k_keys(const double4* __restrict__ pos4, int64_t n,
                                             const GridInfo* __restrict__ gp, uint32_t* __restrict__ keys,
                                             uint32_t* __restrict__ vals) {
  int64_t a = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (a >= n) return;
  const GridInfo& g = *gp;
  double4 p = pos4[a];
  int l = particle_level(p.w, g);
  double c = g.cell[l];
  uint32_t ix = (uint32_t)cell_coord(p.x, g.lo[0], c, g.dims[l][0]);
  uint32_t iy = (uint32_t)cell_coord(p.y, g.lo[1], c, g.dims[l][1]);
  uint32_t iz = (uint32_t)cell_coord(p.z, g.lo[2], c, g.dims[l][2]);
  keys[a] = g.base[l] + (spread3(ix) | (spread3(iy) << 1) | (spread3(iz) << 2));
  vals[a] = (uint32_t)a;
}

// Clears the cells in use (base[nlev] entries) to empty ranges.
__global__ __launch_bounds__(kB) void k_cells_clear(int2* __restrict__ se, const GridInfo* __restrict__ gp) {
  const int64_t total = gp->base[gp->nlev];
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (int64_t)gridDim.x * blockDim.x)
    se[i] = make_int2(0, 0);
}

__global__ __launch_bounds__(kB) void k_cell_ranges(const uint32_t* __restrict__ keys, int64_t n,
                                                    int2* __restrict__ se) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  uint32_t k = keys[i];
  if (i == 0 || keys[i - 1] != k) se[k].x = (int32_t)i;
  if (i == n - 1 || keys[i + 1] != k) se[k].y = (int32_t)(i + 1);
}

// Positions and h in the cell-sorted order (candidate gathers of the build).
__global__ __launch_bounds__(kB) void k_gather_pos(const double4* __restrict__ src, const uint32_t* __restrict__ perm,
                                                   int64_t n, double4* __restrict__ dst) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) dst[i] = src[perm[i]];
}

struct BuildArgs {
  const double4* __restrict__ pos4;
  int64_t n;
  const GridInfo* __restrict__ grid;
  const uint32_t* __restrict__ perm;   // cell-sorted position -> particle index
  const double4* __restrict__ pos_sorted;
  const int2* __restrict__ cell_se;
  const int32_t* __restrict__ tile_start;
  const int32_t* __restrict__ tile_cnt;
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

__device__ __forceinline__ double wave_min_d(double v) {
  for (int off = 32; off > 0; off >>= 1) v = fmin(v, __shfl_xor(v, off, 64));
  return v;
}
__device__ __forceinline__ double wave_max_d(double v) {
  for (int off = 32; off > 0; off >>= 1) v = fmax(v, __shfl_xor(v, off, 64));
  return v;
}
// a value that all lanes hold, in scalar registers
__device__ __forceinline__ double uniform_d(double v) {
  return __hiloint2double(__builtin_amdgcn_readfirstlane(__double2hiint(v)),
                          __builtin_amdgcn_readfirstlane(__double2loint(v)));
}
// min / max over aligned groups of gs lanes (a power of 2, at most 8)
__device__ __forceinline__ double grp_min(double v, int gs) {
  for (int off = 1; off < gs; off <<= 1) v = fmin(v, __shfl_xor(v, off, 64));
  return v;
}
__device__ __forceinline__ double grp_max(double v, int gs) {
  for (int off = 1; off < gs; off <<= 1) v = fmax(v, __shfl_xor(v, off, 64));
  return v;
}
// Geometry of one tile, shared by the cost and build kernels: whole-tile box and max h
// (wave-uniform), and in LDS the sub-boxes of the first 8 groups of gs consecutive particles with their
// own max h.  Candidates and cells are tested against the sub-boxes, which stays tight where a
// tile mixes small and large h (a candidate within (h_a + h_b)(1 + skin) of a particle a is that
// close to a's sub-box).
struct TileGeom {
  double lo[3], hi[3], hmx;
};

__device__ __forceinline__ void tile_geometry(const double4 pa, bool valid, int gs, TileGeom& G, double (*sub)[8]) {
  const int lane = threadIdx.x;
  const double big = 1e300;
  const double q[3] = {pa.x, pa.y, pa.z};
  for (int d = 0; d < 3; ++d) {
    G.lo[d] = uniform_d(wave_min_d(valid ? q[d] : big));
    G.hi[d] = uniform_d(wave_max_d(valid ? q[d] : -big));
  }
  G.hmx = uniform_d(wave_max_d(valid ? pa.w : 0.0));
  double gl[3], gh[3];
  for (int d = 0; d < 3; ++d) {
    gl[d] = grp_min(valid ? q[d] : big, gs);
    gh[d] = grp_max(valid ? q[d] : -big, gs);
  }
  const double gx = grp_max(valid ? pa.w : 0.0, gs);
  const int gi = lane / gs;
  __syncthreads();
  if (gi * gs == lane && gi < 8) {
    for (int d = 0; d < 3; ++d) {
      sub[gi][d] = 0.5 * (gl[d] + gh[d]);
      sub[gi][3 + d] = 0.5 * (gh[d] - gl[d]);
    }
    sub[gi][6] = gx;
  }
  __syncthreads();
}

// Cells of level l that can hold candidates of the tile: the tile box widened by
// (hmx + hlev[l])(1 + skin), clipped to the cells that hold the level's particles.
struct LevelBox {
  int lo3[3], ext[3];
  bool wrap[3];
  int64_t total;
  double c;
  uint32_t base;
};

template <bool PER>
__device__ __forceinline__ bool level_box(const GridInfo& g, int l, const TileGeom& G, double s1, LevelBox& L) {
  if (!g.hlev_bits[l]) return false;   // no particles at this level
  L.c = g.cell[l];
  L.base = g.base[l];
  const double R = (G.hmx + g.hlev[l]) * s1 * (1.0 + 1e-9);
  for (int d = 0; d < 3; ++d) {
    const int dim = g.dims[l][d];
    int l0 = (int)floor((G.lo[d] - R - g.lo[d]) / L.c);
    int h0 = (int)floor((G.hi[d] + R - g.lo[d]) / L.c);
    L.wrap[d] = false;
    if (PER) {
      if (h0 - l0 + 1 >= dim) { l0 = 0; h0 = dim - 1; }
      else L.wrap[d] = true;
    } else {
      const int b0 = cell_coord(dec_double(g.lev_lo[l][d]), g.lo[d], L.c, dim);
      const int b1 = cell_coord(dec_double(g.lev_hi[l][d]), g.lo[d], L.c, dim);
      l0 = l0 < b0 ? b0 : l0;
      h0 = h0 > b1 ? b1 : h0;
    }
    L.lo3[d] = l0;
    L.ext[d] = h0 >= l0 ? h0 - l0 + 1 : 0;
  }
  L.total = (int64_t)L.ext[0] * L.ext[1] * L.ext[2];
  return L.total > 0;
}

// Particle range [s, e) of the cell with linear index j of the level box (empty if the cell is
// farther than (hmax_g + hlev[l])(1 + skin) from every sub-box).  UNR: sub-boxes tested per
// unrolled step (their LDS reads issued together; more registers).
template <bool PER, int UNR>
__device__ __forceinline__ void cell_range(const GridInfo& g, int l, const LevelBox& L, int64_t j, double s1,
                                           const double (*sub)[8], const int2* __restrict__ cell_se, int& s, int& e) {
  s = e = 0;
  if (j >= L.total) return;
  // the box holds at most 2^30 cells (10 bits per axis), so 32-bit index arithmetic suffices
  const unsigned jj = (unsigned)j, e0 = (unsigned)L.ext[0], e1 = (unsigned)L.ext[1];
  const unsigned j1 = jj / e0;
  const int kk[3] = {L.lo3[0] + (int)(jj - j1 * e0), L.lo3[1] + (int)(j1 % e1), L.lo3[2] + (int)(j1 / e1)};
  int cc[3];
  double b0[3], b1[3];
  bool gapd[3];
  for (int d = 0; d < 3; ++d) {
    gapd[d] = !PER || L.wrap[d];
    b0[d] = g.lo[d] + kk[d] * L.c;
    b1[d] = b0[d] + L.c;
    const int dim = g.dims[l][d];
    cc[d] = L.wrap[d] ? ((kk[d] % dim) + dim) % dim : kk[d];
  }
  bool need = false;
#pragma unroll UNR
  for (int gi = 0; gi < 8; ++gi) {
    double gap2 = 0.0;
    for (int d = 0; d < 3; ++d) {
      const double gd = fmax(0.0, fmax(b0[d] - (sub[gi][d] + sub[gi][3 + d]), (sub[gi][d] - sub[gi][3 + d]) - b1[d]));
      gap2 += gapd[d] ? gd * gd : 0.0;
    }
    const double Rg = (sub[gi][6] + g.hlev[l]) * s1 * (1.0 + 1e-9);
    need |= gap2 < Rg * Rg && sub[gi][6] > 0.0;
  }
  if (need) {
    const uint32_t key = L.base + (spread3((uint32_t)cc[0]) | (spread3((uint32_t)cc[1]) << 1) |
                                   (spread3((uint32_t)cc[2]) << 2));
    const int2 se = cell_se[key];
    s = se.x;
    e = se.y;
  }
}

// Cost estimate of each tile: the number of particles in the cells its build would gather.
template <bool PER>
__global__ __launch_bounds__(64) void k_tile_cost(const double4* __restrict__ pos4, const GridInfo* __restrict__ gp,
                                                  const int32_t* __restrict__ tile_start,
                                                  const int32_t* __restrict__ tile_cnt, const int2* __restrict__ cell_se,
                                                  int32_t* __restrict__ cost) {
  __shared__ double sub[8][8];
  const int lane = threadIdx.x;
  const GridInfo& g = *gp;
  const double s1 = 1.0 + g.skin;
  const int64_t ntiles = g.ntiles;
  for (int64_t k_ = blockIdx.x / SPH_XCD, chunk_ = xcd_chunk(ntiles); k_ < chunk_; k_ += gridDim.x / SPH_XCD) {
    const int64_t t = (int64_t)(blockIdx.x % SPH_XCD) * chunk_ + k_;
    if (t >= ntiles) break;
    const bool valid = lane < tile_cnt[t];
    const double4 pa = valid ? pos4[tile_start[t] + lane] : make_double4(0.0, 0.0, 0.0, 0.0);
    TileGeom G;
    tile_geometry(pa, valid, 8, G, sub);
    int64_t tot = 0;
    for (int l = 0; l < g.nlev; ++l) {
      LevelBox L;
      if (!level_box<PER>(g, l, G, s1, L)) continue;
      for (int64_t q = 0; q < L.total; q += 64) {
        int s, e;
        cell_range<PER, 4>(g, l, L, q + lane, s1, sub, cell_se, s, e);
        tot += e - s;
      }
    }
    for (int off = 32; off > 0; off >>= 1) tot += __shfl_xor(tot, off, 64);
    if (lane == 0) cost[t] = (int32_t)(tot < 0x7fffffff ? tot : 0x7fffffff);
    __syncthreads();
  }
}

// Splits expensive tiles: a particle also starts a tile at every 16th (cost > kSplit16 / cdiv) or
// 8th (cost > kSplit8 / cdiv) position of its tile.  The cost counts the particles of the cells a
// build gathers, which shrinks with finer cells (cdiv cells per smoothing diameter).  Reads the
// tile of p from the scan of the old flags.
constexpr int32_t kSplit16 = 12000, kSplit8 = 40000;
__global__ __launch_bounds__(kB) void k_tile_split(uint32_t* __restrict__ flag, const uint32_t* __restrict__ idx,
                                                   int64_t n, const int32_t* __restrict__ tile_start,
                                                   const int32_t* __restrict__ cost, int cdiv,
                                                   uint32_t* __restrict__ bsum) {
  __shared__ uint32_t tot;
  const int64_t p0 = (int64_t)blockIdx.x * 1024 + threadIdx.x * 4;
  if (threadIdx.x == 0) tot = 0u;
  __syncthreads();
  uint32_t v = 0u;
  for (int k = 0; k < 4; ++k) {
    const int64_t p = p0 + k;
    if (p >= n) break;
    const uint32_t f = flag[p];
    const int64_t t = (int64_t)idx[p] + f - 1;
    const int32_t c = cost[t];
    const int64_t off = p - tile_start[t];
    const int size = c > kSplit8 / cdiv ? 8 : (c > kSplit16 / cdiv ? 16 : 64);
    const uint32_t g = (f || (off % size) == 0) ? 1u : 0u;
    flag[p] = g;
    v += g;
  }
  atomicAdd(&tot, v);
  __syncthreads();
  if (threadIdx.x == 0) bsum[blockIdx.x] = tot;   // starts per block of 1024 particles
}

// Tile neighbour lists.  Each tile is handled by one wavefront (one lane per target), in three
// latency-friendly phases per block of 64 candidate cells:
//  1. the 64 lanes take 64 cells of the level box at once, cull them against the sub-boxes and
//     load their particle ranges;
//  2. the wave gathers the cells' particles 64 at a time (a wave-wide prefix sum maps lanes to
//     (cell, offset)), tests each against the tile's box and appends survivors to an LDS batch;
//  3. a batch of 64 candidates is tested against the 64 targets on the matrix cores (sph_build.h):
//     the sign of r^2 - (h_a' + h_b')^2 is the decision wherever its size exceeds kBand (|x|^2 + h'^2
//     of both), twice what the test can be off (16 2^-22 of that, see the other build's bound); the few
//     pairs within it are decided by the FP64 test.
// The decision is thus the FP64 one for every pair, r^2 < (h_a' + h_b')^2 with h' = h (1 + skin)
// (1 + 2^-40) and r^2 by FMA: the factor 1 + 2^-40 exceeds the few ulp by which this rounding can differ
// from the exact decision of the density pass, so the candidates always contain every pair that test can
// accept (with a positive skin the rebuild test's own margin of 1e-9 is larger still).
// Tile t is particles [tile_start[t], tile_start[t] + tile_cnt[t]) of the array order (at most 64).
// Candidates enter batches in a fixed order (level, cell, cell-sorted position); one that any target
// hits joins the union, as its next member, and each target appends the local indices of its hits, so U
// and the lists are deterministic and each list is ascending in local index.
// Bound by instruction issue.  The FP64 test of every candidate by every lane (10 operations a pair, and
// eight sub-box tests a candidate to keep the batches short) took 3.43 ms on the 2M star (skin 0.14),
// 1.08 ms on a 300k snapshot and 0.50 ms on the 1M shell; this takes 1.88, 0.51 and
// 0.32.  (Sub-box or particle tests of the candidates on top of the box test cost more than the batches
// they save: 3.11 ms with the sub-boxes, 2.27 against 2.15 with the particles of small tiles.)
constexpr float kBand = 0x1p-17f;
template <bool PER, int NL>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(3))) void k_build_tiles(BuildArgs B) {
  __shared__ int32_t c_s[64], c_o[64];
  __shared__ double sub[8][8];   // per group of 8 tile particles: centre xyz, half-width xyz, max h
  __shared__ float4 cb[128];     // candidates waiting: scaled x, y, z, h'
  __shared__ int32_t cbi[128];
  __shared__ __align__(16) uint16_t ring[64 * kRingRow];
  // a batch's candidate that is target l itself, in the padding of its ring
  auto self = [&](int l) -> uint32_t& { return *reinterpret_cast<uint32_t*>(ring + kRingRow * l + kRing); };
  const int lane = threadIdx.x;
  const unsigned long long lt = lane ? (~0ull >> (64 - lane)) : 0ull;
  const GridInfo& g = *B.grid;
  const double box = g.box;
  const double s1 = 1.0 + g.skin;
  const double s1w = s1 * (1.0 + 0x1p-40);   // the batch test's widened factor
  // the candidate of a batch that this lane lifts: the products' rows come out in an order in which
  // lane l holds bit l' of the masks, so it takes candidate l' and the bits are in batch order
  const int lj = 32 * ((lane >> 2) & 1) + 16 * (lane >> 5) + 4 * ((lane >> 3) & 3) + (lane & 3);
  const int64_t ntiles = g.ntiles;
  for (int64_t k_ = blockIdx.x / SPH_XCD, chunk_ = xcd_chunk(ntiles); k_ < chunk_; k_ += gridDim.x / SPH_XCD) {
    const int64_t t = (int64_t)(blockIdx.x % SPH_XCD) * chunk_ + k_;
    if (t >= ntiles) break;
    const int32_t tcnt = B.tile_cnt[t], ts = B.tile_start[t];
    const bool valid = lane < tcnt;
    const int32_t a = ts + lane;
    const double4 pa = valid ? B.pos4[a] : make_double4(0.0, 0.0, 0.0, 0.0);
    const double ha = pa.w * s1w;
    TileGeom G;
    // small tiles (split off because their neighbourhoods are dear) are often a few particles far apart:
    // cells are culled against groups as small as 8 boxes allow, down to the single particle
    tile_geometry(pa, valid, tcnt > 32 ? 8 : (tcnt > 16 ? 4 : (tcnt > 8 ? 2 : 1)), G, sub);
    const double cx = uniform_d(0.5 * (G.lo[0] + G.hi[0])), cy = uniform_d(0.5 * (G.lo[1] + G.hi[1])),
                 cz = uniform_d(0.5 * (G.lo[2] + G.hi[2]));
    const double wx = uniform_d(0.5 * (G.hi[0] - G.lo[0])), wy = uniform_d(0.5 * (G.hi[1] - G.lo[1])),
                 wz = uniform_d(0.5 * (G.hi[2] - G.lo[2]));
    const uint32_t uoff = B.tile_uoff[t];
    int ucap = (int)((int64_t)tcnt * B.cap < B.ucap ? (int64_t)tcnt * B.cap : B.ucap);
    if ((int64_t)uoff + ucap > B.upool) {
      ucap = 0;
      if (lane == 0) latch_error(B.status, SPH_E_NGB_CAPACITY, -1);
    }
    int32_t* U = B.tile_u + uoff;
    // lengths are scaled so that the tile's reach is 100 (in FP64, whatever the caller's unit of length)
    const double wr = uniform_d(sqrt(wx * wx + wy * wy + wz * wz)), hr = uniform_d(G.hmx * s1);
    const double sc = uniform_d(100.0 / (wr + 2.0 * hr + 1e-290));
    const float reach = (float)((wr + hr) * sc) * (1.f + 1e-4f);
    // scaled components of a particle at d from the tile's centre
    auto scaled = [&](double dx, double dy, double dz, double hp) {
      return make_float4((float)(dx * sc), (float)(dy * sc), (float)(dz * sc), (float)(hp * sc));
    };
    // the lane's particle of a product; one that is not there or out of every target's reach never hits.
    // Returns |x|^2 + h'^2
    auto lift = [&](float4& p, bool in, float& w) -> float {
      const float r2 = p.x * p.x + p.y * p.y + p.z * p.z, h2 = p.w * p.w, far = reach + p.w;
      w = r2 - h2;
      if (!(in && r2 < far * far && h2 < 1e30f)) {   // (NaN fails too)
        p = make_float4(0.f, 0.f, 0.f, 0.f);
        w = 60000.f;
        return 0.f;
      }
      return r2 + h2;
    };
    constexpr float kListMax = 3e4f;   // |x|^2 + h'^2 that FP16 takes
    f16x8 T[2];
    bool by_pair;
    {
      float w;
      float4 p = scaled(min_image(pa.x - cx, (int)PER, box), min_image(pa.y - cy, (int)PER, box),
                        min_image(pa.z - cz, (int)PER, box), ha);
      const float m = lift(p, valid, w);
      lift_operands<true>(p.x, p.y, p.z, p.w, w, T);
      by_pair = __ballot(m > 0.5f * kListMax) != 0ull;
    }
    // a periodic box less than twice the reach across: images of a pair relative to the centre may differ
    if (PER) by_pair = by_pair || fmax(wx, fmax(wy, wz)) + (G.hmx + g.hmax) * s1 * (1.0 + 1e-5) > 0.499 * box;
    ListOut<NL> out;
    out.ring = ring + kRingRow * lane;
    out.slot0 = reinterpret_cast<uint4*>(B.nbr16) + (valid ? (int64_t)a : 0) * NL;
    out.gstride = B.capw * NL;
    out.cap_sl = B.cap_sl;
    out.cnt = out.stored = 0;
    int usize = 0;
    // the FP64 decision of the lane's target on a waiting candidate
    auto exact = [&](int j) -> bool {
      const double4 q = B.pos4[cbi[j]];
      const double dx = min_image(pa.x - q.x, (int)PER, box), dy = min_image(pa.y - q.y, (int)PER, box),
                   dz = min_image(pa.z - q.z, (int)PER, box);
      const double H = ha + q.w * s1w;
      return fma(dz, dz, fma(dy, dy, dx * dx)) < H * H;
    };
    auto batch = [&](int nb) {
      const bool in = lj < nb;
      float4 p = cb[lj];
      const int32_t b = in ? cbi[lj] : -1;
      uint32_t m0, m1;
      float w;
      const float mag = lift(p, in, w);
      if (!by_pair && !__ballot(mag > kListMax)) {
        f16x8 C[2];
        lift_operands<false>(p.x, p.y, p.z, p.w, w, C);
        const float band = kBand * (0.5f * kListMax + (__ballot(mag > 0.5f * kListMax) ? kListMax : 0.5f * kListMax));
        uint32_t q[2], near[2] = {0u, 0u};
#pragma unroll
        for (int tb = 0; tb < 2; ++tb) {
          __builtin_amdgcn_sched_barrier(0);   // 32 of the products' registers at a time
          const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
          const f32x16 D0 = __builtin_amdgcn_mfma_f32_32x32x16_f16(C[0], T[tb], zero, 0, 0, 0);
          const f32x16 D1 = __builtin_amdgcn_mfma_f32_32x32x16_f16(C[1], T[tb], zero, 0, 0, 0);
          uint32_t q0 = 0u, q1 = 0u;
          float least = 1e30f;
#pragma unroll
          for (int e = 15; e >= 0; --e) {
            q0 = __builtin_amdgcn_alignbit(q0, __float_as_uint(D0[e]), 31u);
            q1 = __builtin_amdgcn_alignbit(q1, __float_as_uint(D1[e]), 31u);
            least = fminf(fminf(least, fabsf(D0[e])), fabsf(D1[e]));
          }
          q[tb] = q0 | (q1 << 16);
          if (__ballot(least < band)) {
            uint32_t n0 = 0u, n1 = 0u;
#pragma unroll
            for (int e = 15; e >= 0; --e) {
              n0 = __builtin_amdgcn_alignbit(n0, __float_as_uint(fabsf(D0[e]) - band), 31u);
              n1 = __builtin_amdgcn_alignbit(n1, __float_as_uint(fabsf(D1[e]) - band), 31u);
            }
            near[tb] = n0 | (n1 << 16);
          }
        }
        // lane l < 32 holds rows 8 i + j (upper lanes: 8 i + 4 + j) of targets l and 32 + l: each
        // lane receives both halves of its own target
        m0 = q[0];
        m1 = q[1];
        swap32(m0, m1);
        if (__ballot((near[0] | near[1]) != 0u)) {
          swap32(near[0], near[1]);
          auto decide = [&](uint32_t m, uint32_t left, int base) -> uint32_t {
            while (left) {
              const int k = __builtin_ctz(left);
              left &= left - 1;
              m = (m & ~(1u << k)) | ((exact(base + k) ? 1u : 0u) << k);
            }
            return m;
          };
          m0 = decide(m0, near[0], 0);
          m1 = decide(m1, near[1], 32);
        }
      } else {
        m0 = m1 = 0u;
        for (int j = 0; j < nb; ++j) {
          const uint32_t bit = (valid && exact(j) ? 1u : 0u) << (j & 31);
          if (j < 32) m0 |= bit;
          else m1 |= bit;
        }
      }
      // a particle is not its own neighbour
      const int ta = b - ts;   // the target this candidate is, if it is of the tile
      if (__ballot(in && ta >= 0 && ta < tcnt)) {
        self(lane) = 64u;
        __syncthreads();
        if (in && ta >= 0 && ta < tcnt) self(ta) = (uint32_t)lj;
        __syncthreads();
        const uint32_t sb = self(lane);
        if (sb < 32u) m0 &= ~(1u << sb);
        else if (sb < 64u) m1 &= ~(1u << (sb - 32u));
      }
      const uint32_t u0 = wave_or(m0), u1 = wave_or(m1);   // the batch's union members
      if (!(u0 | u1)) return;
      const int n0 = __builtin_popcount(u0);
      {
        const uint32_t uw = lj < 32 ? u0 : u1;
        const int loc = usize + (lj < 32 ? 0 : n0) + __builtin_popcount(uw & ((1u << (lj & 31)) - 1u));
        if (((uw >> (lj & 31)) & 1u) && loc < ucap) U[loc] = b;
      }
      out.append(m0, m1, u0, u1, usize, ucap > 0 ? ucap - 1 : 0);
      usize += n0 + __builtin_popcount(u1);
    };
    int pend = 0;   // candidates waiting in cb (wave-uniform)
    for (int l = 0; l < g.nlev; ++l) {
      LevelBox L;
      if (!level_box<PER>(g, l, G, s1, L)) continue;
      for (int64_t q = 0; q < L.total; q += 64) {
        // phase 1: 64 cells at once; lanes take the block's cells in bit-reversed order so that
        // consecutive union members come from all over the neighbourhood and every target's
        // neighbours spread evenly over the LDS chunks of the pair passes
        int s, e;
        cell_range<PER, 2>(g, l, L, q + (int64_t)(__brev((unsigned)lane) >> 26), s1, sub, B.cell_se, s, e);
        // wave prefix sum of the cells' particle counts
        const int cntc = e - s;
        int inc = cntc;
        for (int off = 1; off < 64; off <<= 1) {
          const int o = __shfl_up(inc, off, 64);
          if (lane >= off) inc += o;
        }
        const int Tc = __shfl(inc, 63, 64);
        __syncthreads();
        // the cells with particles, in order: the end of each in the block's candidates, and what leads from
        // a candidate to its cell-sorted position
        const unsigned long long filled = __ballot(cntc > 0);
        if (cntc > 0) {
          const int k = __popcll(filled & lt);
          c_s[k] = s - (inc - cntc);
          c_o[k] = inc;
        }
        __syncthreads();
        // phase 2: gather candidates 64 at a time, the next 64 in flight, test against the tile's box
        // and append the survivors to the batch in slot order
        // (a lane's candidates ascend, so it goes on from its last cell: a binary search of the block in
        // every round is six dependent LDS reads, 2.15 instead of 1.88 ms on the 2M star)
        int cell = -1, cend = 0, cbase = 0;
        auto fetch = [&](int slot, double4& pb) -> int32_t {
          pb = make_double4(0.0, 0.0, 0.0, 0.0);
          if (slot >= Tc) return -1;
          while (slot >= cend) {   // ends: the last filled cell ends at Tc
            ++cell;
            cbase = c_s[cell];
            cend = c_o[cell];
          }
          const int32_t sp = cbase + slot;
          pb = B.pos_sorted[sp];
          return (int32_t)B.perm[sp];
        };
        double4 p0;
        int32_t b0 = fetch(lane, p0);
#pragma unroll 1
        for (int q0 = 0; q0 < Tc; q0 += 64) {
          double4 p1;
          const int32_t b1 = fetch(q0 + 64 + lane, p1);
          const double dx = min_image(p0.x - cx, (int)PER, box), dy = min_image(p0.y - cy, (int)PER, box),
                       dz = min_image(p0.z - cz, (int)PER, box);
          const double ex = fmax(0.0, fabs(dx) - wx), ey = fmax(0.0, fabs(dy) - wy), ez = fmax(0.0, fabs(dz) - wz);
          const double Rb = (G.hmx + p0.w) * s1 * (1.0 + 1e-9);
          const bool pass = b0 >= 0 && ex * ex + ey * ey + ez * ez < Rb * Rb;
          const unsigned long long m = __ballot(pass);
          if (pass) {
            const int k = pend + __popcll(m & lt);
            cb[k] = scaled(dx, dy, dz, p0.w * s1w);
            cbi[k] = b0;
          }
          pend += __popcll(m);
          __syncthreads();
          if (pend >= 64) {   // phase 3 on a full batch
            batch(64);
            const int rest = pend - 64;
            float4 mv = make_float4(0.f, 0.f, 0.f, 0.f);
            int32_t mi = 0;
            if (lane < rest) { mv = cb[64 + lane]; mi = cbi[64 + lane]; }
            __syncthreads();
            if (lane < rest) { cb[lane] = mv; cbi[lane] = mi; }
            pend = rest;
            __syncthreads();
          }
          p0 = p1;
          b0 = b1;
        }
      }
    }
    if (pend > 0) batch(pend);
    __syncthreads();
    if (valid) out.finish();
    if (valid) B.count[a] = out.cnt < B.cap ? out.cnt : B.cap;
    if (lane == 0) B.tile_usize[t] = usize < ucap ? usize : ucap;
    if (usize > ucap || out.cnt > B.cap) latch_error(B.status, SPH_E_NGB_CAPACITY, valid ? a : -1);
  }
}

// Cells per smoothing diameter of the finest level (default 1: cells of 2 hmax_l).  Measured on
// the 2M-particle star, 1 against 2 takes a list build from 6.2 to 5.3 ms (8x fewer cells to
// cull, at 1.5x more particles to pre-test) and the FP32 step from 1.335 to 1.288 ms.
static int cell_div_of(const sph_params& p) { return p.cell_div > 0 ? p.cell_div : 1; }

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

}  // namespace

// Grid, cell-sorted order and cell ranges of the current pos4 (overwrites keys and vals).
sph_status grid_prepare(sph_ctx* c, int64_t n) {
  hipStream_t s = c->stream;
  const unsigned nb = grid_for(n, kB), nred = nb < 512 ? nb : 512;
  sph_status e;
  hipLaunchKernelGGL(k_level_hmax, dim3(nred), dim3(kB), 0, s, c->pos4, n, c->grid);
  hipLaunchKernelGGL(k_grid_setup2, dim3(1), dim3(1), 0, s, c->grid, cell_div_of(c->p),
                     c->max_cells, c->status);
  hipLaunchKernelGGL(k_keys, dim3(nb), dim3(kB), 0, s, c->pos4, n, c->grid, c->keys, c->vals);
  if ((e = sph_sort_pairs(c, c->keys, c->vals, n))) return e;
  hipLaunchKernelGGL(k_cells_clear, dim3(2048), dim3(kB), 0, s, c->cell_se, c->grid);
  hipLaunchKernelGGL(k_cell_ranges, dim3(nb), dim3(kB), 0, s, c->keys, n, c->cell_se);
  hipLaunchKernelGGL(k_gather_pos, dim3(nb), dim3(kB), 0, s, c->pos4, c->vals, n, c->pos_sorted);
  HIP_TRY(hipGetLastError());
  return SPH_OK;
}

// Marks the starts of the tiles that the cost estimate splits off in flag (idx: its scan so far);
// bsum: the starts per block of 1024 particles.
sph_status grid_split_tiles(sph_ctx* c, int64_t n, uint32_t* flag, const uint32_t* idx, unsigned tiles, uint32_t* bsum) {
  if (c->p.periodic)
    hipLaunchKernelGGL(HIP_KERNEL_NAME(k_tile_cost<true>), dim3(tiles), dim3(64), 0, c->stream, c->pos4, c->grid,
                       c->tile_start, c->tile_cnt, c->cell_se, c->tile_usize);
  else
    hipLaunchKernelGGL(HIP_KERNEL_NAME(k_tile_cost<false>), dim3(tiles), dim3(64), 0, c->stream, c->pos4, c->grid,
                       c->tile_start, c->tile_cnt, c->cell_se, c->tile_usize);
  hipLaunchKernelGGL(k_tile_split, dim3(grid_for(n, 1024)), dim3(kB), 0, c->stream, flag, idx, n, c->tile_start,
                     c->tile_usize, cell_div_of(c->p), bsum);
  HIP_TRY(hipGetLastError());
  return SPH_OK;
}

sph_status grid_build_lists(sph_ctx* c, int64_t n, unsigned tiles) {
  BuildArgs B;
  B.pos4 = c->pos4; B.n = n; B.grid = c->grid; B.perm = c->vals; B.pos_sorted = c->pos_sorted;
  B.cell_se = c->cell_se; B.capw = c->capw; B.cap = c->cap_s; B.ucap = c->ucap;
  B.lanes = pass_lanes(c->p); B.cap_sl = cand_slot_capacity(c->cap_s, B.lanes);
  B.tile_start = c->tile_start; B.tile_cnt = c->tile_cnt; B.tile_uoff = c->tile_uoff; B.upool = c->upool;
  B.tile_u = c->tile_u; B.tile_usize = c->tile_usize; B.nbr16 = c->nbr16s; B.count = c->nbr_count_s;
  B.status = c->status;
  launch_build(B, c->p.periodic != 0, dim3(tiles), c->stream);
  HIP_TRY(hipGetLastError());
  return SPH_OK;
}
