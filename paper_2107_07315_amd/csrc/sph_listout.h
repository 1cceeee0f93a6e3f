// A target's candidate list in the making (sph_build.h).  Plain enough to be compiled for the host, where
// its store is tested.
#pragma once
#include <stdint.h>

namespace {

// A target's list in the making.  Candidate k of a particle goes to its slot k % L, as entry k / L
// (L = lanes per target of the pair passes).  Hits wait in the lane's LDS ring of 64 entries in
// arrival order; 8 L of them are one group of 8 entries of every slot, gathered from the ring by
// byte permutes and stored as L 16-byte groups (group g of slot s at g * capw * L + s).
constexpr int kRing = 64, kRingRow = 72;   // ring entries, and the padded row (16-byte aligned)
template <int L>
struct ListOut {
  uint16_t* ring;
  uint4* slot0;       // group 0 of the target's first slot
  int64_t gstride;    // groups between consecutive groups of one slot (capw * L)
  int cap_sl;
  int cnt, stored;    // hits so far, groups stored
  __device__ __forceinline__ void store_group(int nslots) {
    uint32_t D[4 * L];
    __builtin_memcpy(D, __builtin_assume_aligned(ring + ((8 * L * stored) & (kRing - 1)), 16), sizeof(D));
#pragma unroll
    for (int s = 0; s < L; ++s) {
      if (s >= nslots) break;
      uint32_t w[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        if constexpr (L == 1) {
          w[k] = D[k];
        } else {
          const int i0 = 2 * k * L + s, i1 = (2 * k + 1) * L + s;   // entries 2k, 2k + 1 of slot s
          const uint32_t sel = ((i0 & 1) ? 0x0302u : 0x0100u) | ((i1 & 1) ? 0x07060000u : 0x05040000u);
          w[k] = __builtin_amdgcn_perm(D[i1 >> 1], D[i0 >> 1], sel);
        }
      }
      if (stored * 8 < cap_sl) slot0[(int64_t)stored * gstride + s] = make_uint4(w[0], w[1], w[2], w[3]);
    }
    ++stored;
  }
  // room for `more` entries in every lane's ring (the wave's complete groups are stored if not)
  __device__ __forceinline__ void make_room(int more) {
    if (__ballot(cnt - 8 * L * stored + more > kRing))
      while (cnt - 8 * L * stored >= 8 * L) store_group(L);
  }
  // the lowest hit left in m, entry k: bit b is union member base + (members of um below b)
  __device__ __forceinline__ void put(uint32_t& m, uint32_t um, int base, int last, int k) {
    const int b = __builtin_ctz(m);
    m &= m - 1;
    int loc = base + __builtin_popcount(um & ((1u << b) - 1u));
    loc = loc < last ? loc : last;   // union overflow: keep reads in range, error latched
    const uint16_t v = (uint16_t)loc;
    __builtin_memcpy(ring + (k & (kRing - 1)), &v, sizeof(v));
  }
  // the hits of a batch: words m0 (members from base of u0) and m1 (after them, of u1); both words
  // advance together where the ring holds them
  __device__ __forceinline__ void append(uint32_t m0, uint32_t m1, uint32_t u0, uint32_t u1, int base, int last) {
    const int n0 = __builtin_popcount(m0), nn = n0 + __builtin_popcount(m1), base1 = base + __builtin_popcount(u0);
    make_room(nn);
    if (!__ballot(cnt - 8 * L * stored + nn > kRing)) {
      int k = cnt;
      while (m0 | m1) {
        if (m0) put(m0, u0, base, last, k);
        if (m1) put(m1, u1, base1, last, k + n0);
        ++k;
      }
    } else {
      make_room(n0);
      for (int k = cnt; m0; ++k) put(m0, u0, base, last, k);
      cnt += n0;
      make_room(nn - n0);
      for (int k = cnt; m1; ++k) put(m1, u1, base1, last, k);
      cnt -= n0;
    }
    cnt += nn;
  }
  // The entries left in the ring: whole groups, then a partly filled last one (slots s < r of it hold
  // entries).  A list past its capacity too: the passes walk the entries that it counts, the first ones up
  // to the capacity, even though the error is latched, so each of them has to be there.
  __device__ __forceinline__ void finish() {
    while (cnt - 8 * L * stored >= 8 * L) store_group(L);
    const int r = cnt - 8 * L * stored;
    if (r > 0) store_group(r < L ? r : L);
  }
};

}  // namespace
