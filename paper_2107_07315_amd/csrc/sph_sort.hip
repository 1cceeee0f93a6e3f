// Stable LSD radix sort of (32-bit key, 32-bit value) pairs, 8-bit digits, for the list builds.
// Per pass: block histograms -> exclusive scan over (digit, block) in two small kernels (for small sets
// within the scatter) -> stable scatter.  The
// scatter ranks keys inside a 64-lane wave with ballot-based digit matching and orders waves and
// rounds through LDS counters, so equal keys keep their input order.
#include "sph_internal.h"

namespace {

constexpr int kBlock = 256;             // 4 waves of 64
constexpr int kItems = 16;              // keys per thread per tile
constexpr int kTile = kBlock * kItems;  // 4096 keys per block

__global__ __launch_bounds__(kBlock) void k_hist(const uint32_t* __restrict__ keys, int64_t n, int shift,
                                                 uint32_t* __restrict__ hist, int nblocks) {
  __shared__ uint32_t h[256];
  h[threadIdx.x] = 0;
  __syncthreads();
  int64_t base = (int64_t)blockIdx.x * kTile;
  for (int r = 0; r < kItems; ++r) {
    int64_t i = base + (int64_t)r * kBlock + threadIdx.x;
    if (i < n) atomicAdd(&h[(keys[i] >> shift) & 255u], 1u);
  }
  __syncthreads();
  hist[(int64_t)threadIdx.x * nblocks + blockIdx.x] = h[threadIdx.x];
}

// Block-wide exclusive scan of one value per thread (256 threads = 4 waves).
__device__ __forceinline__ uint32_t block_exclusive_scan(uint32_t v, uint32_t* wsum, uint32_t& total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint32_t inc = v;
  for (int off = 1; off < 64; off <<= 1) {
    uint32_t o = __shfl_up(inc, off, 64);
    if (lane >= off) inc += o;
  }
  if (lane == 63) wsum[wave] = inc;
  __syncthreads();
  uint32_t before = 0;
  for (int w = 0; w < wave; ++w) before += wsum[w];
  total = wsum[0] + wsum[1] + wsum[2] + wsum[3];
  __syncthreads();
  return before + inc - v;
}

// Row scan: block d turns hist[d][0..nblocks) into exclusive prefixes and stores the row total.
__global__ __launch_bounds__(256) void k_scan_rows(uint32_t* __restrict__ hist, int nblocks,
                                                   uint32_t* __restrict__ rowtot) {
  __shared__ uint32_t wsum[4];
  uint32_t* row = hist + (int64_t)blockIdx.x * nblocks;
  uint32_t carry = 0;
  for (int base = 0; base < nblocks; base += 256) {
    int i = base + threadIdx.x;
    uint32_t v = i < nblocks ? row[i] : 0u;
    uint32_t tot;
    uint32_t ex = block_exclusive_scan(v, wsum, tot);
    if (i < nblocks) row[i] = carry + ex;
    carry += tot;
  }
  if (threadIdx.x == 0) rowtot[blockIdx.x] = carry;
}

// Exclusive scan of the 256 row totals (digit offsets).
__global__ __launch_bounds__(256) void k_scan_totals(uint32_t* __restrict__ rowtot) {
  __shared__ uint32_t wsum[4];
  uint32_t tot;
  uint32_t v = rowtot[threadIdx.x];
  uint32_t ex = block_exclusive_scan(v, wsum, tot);
  rowtot[threadIdx.x] = ex;
}

// One round of a block's scatter: 256 keys, ranked inside each wave by digit matching, after the keys
// of earlier rounds (base) and of the block's earlier waves (wave_cnt).
__device__ __forceinline__ void scatter_round(int64_t i, int64_t n, int shift, int lane, int wave,
                                              const uint32_t* __restrict__ keys, const uint32_t* __restrict__ vals,
                                              uint32_t* base, uint32_t (*wave_cnt)[256], uint32_t* __restrict__ keys_out,
                                              uint32_t* __restrict__ vals_out) {
  const unsigned long long lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
  bool valid = i < n;
  uint32_t k = valid ? keys[i] : 0u;
  uint32_t v = valid ? vals[i] : 0u;
  uint32_t d = (k >> shift) & 255u;
  // lanes holding the same digit
  unsigned long long match = __ballot(valid);
  for (int b = 0; b < 8; ++b) {
    unsigned long long bb = __ballot((d >> b) & 1u);
    match &= ((d >> b) & 1u) ? bb : ~bb;
  }
  uint32_t rank = (uint32_t)__popcll(match & lt);
  bool leader = valid && ((match & lt) == 0ull);
  if (leader) wave_cnt[wave][d] = (uint32_t)__popcll(match);
  __syncthreads();
  if (valid) {
    uint32_t pos = base[d] + rank;
    for (int w = 0; w < wave; ++w) pos += wave_cnt[w][d];
    keys_out[pos] = k;
    vals_out[pos] = v;
  }
  __syncthreads();
  // advance the per-digit base by this round's total and clear the wave counters
  uint32_t tot = 0;
  for (int w = 0; w < 4; ++w) {
    tot += wave_cnt[w][threadIdx.x];
    wave_cnt[w][threadIdx.x] = 0;
  }
  base[threadIdx.x] += tot;
  __syncthreads();
}

__global__ __launch_bounds__(kBlock) void k_scatter(const uint32_t* __restrict__ keys,
                                                    const uint32_t* __restrict__ vals, int64_t n,
                                                    int shift, const uint32_t* __restrict__ offs,
                                                    const uint32_t* __restrict__ digit_off,
                                                    int nblocks, uint32_t* __restrict__ keys_out,
                                                    uint32_t* __restrict__ vals_out) {
  __shared__ uint32_t base[256];
  __shared__ uint32_t wave_cnt[4][256];
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  base[threadIdx.x] = digit_off[threadIdx.x] + offs[(int64_t)threadIdx.x * nblocks + blockIdx.x];
  for (int w = 0; w < 4; ++w) wave_cnt[w][threadIdx.x] = 0;
  __syncthreads();
  int64_t tile0 = (int64_t)blockIdx.x * kTile;
  for (int r = 0; r < kItems; ++r)
    scatter_round(tile0 + (int64_t)r * kBlock + threadIdx.x, n, shift, lane, wave, keys, vals, base, wave_cnt, keys_out,
                  vals_out);
}

// Up to kSmallBlocks blocks of 1024 keys: the same pass with a quarter of the keys a block (a pass is
// a chain of rounds of 256 keys) and the offsets summed by each block from the histogram itself, so a
// pass is two launches: at 20k particles 8 launches of 4 us instead of 16 of 6 us a sort.
constexpr int kSmallItems = 4, kSmallTile = kBlock * kSmallItems, kSmallBlocks = 128;
__global__ __launch_bounds__(kBlock) void k_hist_small(const uint32_t* __restrict__ keys, int64_t n, int shift,
                                                       uint32_t* __restrict__ hist) {
  __shared__ uint32_t h[256];
  h[threadIdx.x] = 0;
  __syncthreads();
  const int64_t base = (int64_t)blockIdx.x * kSmallTile;
  for (int r = 0; r < kSmallItems; ++r) {
    const int64_t i = base + (int64_t)r * kBlock + threadIdx.x;
    if (i < n) atomicAdd(&h[(keys[i] >> shift) & 255u], 1u);
  }
  __syncthreads();
  hist[(int64_t)blockIdx.x * 256 + threadIdx.x] = h[threadIdx.x];
}
__global__ __launch_bounds__(kBlock) void k_scatter_small(const uint32_t* __restrict__ keys,
                                                          const uint32_t* __restrict__ vals, int64_t n, int shift,
                                                          const uint32_t* __restrict__ hist, int nblocks,
                                                          uint32_t* __restrict__ keys_out, uint32_t* __restrict__ vals_out) {
  __shared__ uint32_t base[256];
  __shared__ uint32_t wave_cnt[4][256];
  __shared__ uint32_t wsum[4];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint32_t before = 0, all = 0, tot;   // this thread's digit: in earlier blocks, in all blocks
  for (int b = 0; b < nblocks; ++b) {
    const uint32_t v = hist[(int64_t)b * 256 + threadIdx.x];
    all += v;
    before += b < (int)blockIdx.x ? v : 0u;
  }
  base[threadIdx.x] = block_exclusive_scan(all, wsum, tot) + before;
  for (int w = 0; w < 4; ++w) wave_cnt[w][threadIdx.x] = 0;
  __syncthreads();
  const int64_t tile0 = (int64_t)blockIdx.x * kSmallTile;
  for (int r = 0; r < kSmallItems; ++r)
    scatter_round(tile0 + (int64_t)r * kBlock + threadIdx.x, n, shift, lane, wave, keys, vals, base, wave_cnt, keys_out,
                  vals_out);
}

}  // namespace

void sph_scan_rows(sph_ctx* c, uint32_t* v, int nb, uint32_t* total, int rows) {
  hipLaunchKernelGGL(k_scan_rows, dim3((unsigned)rows), dim3(256), 0, c->stream, v, nb, total);
}

// Sorts keys[0..n) ascending, carrying vals; on return keys/vals hold the sorted pairs.
sph_status sph_sort_pairs(sph_ctx* c, uint32_t* keys, uint32_t* vals, int64_t n) {
  if (n <= 1) return SPH_OK;
  int nblocks = (int)((n + kTile - 1) / kTile);
  if (nblocks > c->sort.max_blocks) return SPH_E_ARG;
  const int nsmall = (int)((n + kSmallTile - 1) / kSmallTile);
  uint32_t *ka = keys, *va = vals, *kb = c->sort.keys_alt, *vb = c->sort.vals_alt;
  for (int shift = 0; shift < 32; shift += 8) {
    if (nsmall <= kSmallBlocks) {
      hipLaunchKernelGGL(k_hist_small, dim3(nsmall), dim3(kBlock), 0, c->stream, ka, n, shift, c->sort.hist);
      hipLaunchKernelGGL(k_scatter_small, dim3(nsmall), dim3(kBlock), 0, c->stream, ka, va, n, shift, c->sort.hist, nsmall,
                         kb, vb);
    } else {
      hipLaunchKernelGGL(k_hist, dim3(nblocks), dim3(kBlock), 0, c->stream, ka, n, shift, c->sort.hist,
                         nblocks);
      hipLaunchKernelGGL(k_scan_rows, dim3(256), dim3(256), 0, c->stream, c->sort.hist, nblocks, c->sort.rowtot);
      hipLaunchKernelGGL(k_scan_totals, dim3(1), dim3(256), 0, c->stream, c->sort.rowtot);
      hipLaunchKernelGGL(k_scatter, dim3(nblocks), dim3(kBlock), 0, c->stream, ka, va, n, shift,
                         c->sort.hist, c->sort.rowtot, nblocks, kb, vb);
    }
    uint32_t* t = ka; ka = kb; kb = t;
    t = va; va = vb; vb = t;
  }
  // four passes: the result is back in the caller's buffers
  HIP_TRY(hipGetLastError());
  return SPH_OK;
}
