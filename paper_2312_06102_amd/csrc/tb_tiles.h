// tb_tiles.h -- per-tile cell counting shared by the reorder pass and the block
// builder: a particle i that starts cells at depths A_i .. D_i (A_i > D_i: none)
// adds one cell to each of those depths; per-thread counts are packed two
// 16-bit depths to a word and scanned across the workgroup.
#pragma once

#include "tb_internal.h"

namespace tb {

constexpr int kWaves = kCellThreads / 64;

#if defined(__HIP_DEVICE_COMPILE__) || defined(__HIPCC__)

// Per-thread packed per-depth counts of the cells started by this thread's
// particles (particle i starts the cells at depths A_i .. D_i).  The particles' depth
// masks are added bit-sliced (bit d of plane k: bit k of depth d's count); the words of
// depths that no particle of the wave starts a cell at are 0 without further work (a
// tile of 2^24 random particles has cells at 4 or 5 of the 22 depths; with every depth of
// every particle compared this and the scan below were 0.3 of the instructions of the
// emit pass: 2^24 clustered particles 283 us, 255 us now).
template <int IPT>
__device__ inline void thread_level_counts(const uint8_t (&A)[IPT], const uint8_t (&D)[IPT],
                                           uint32_t c[kLevelWords]) {
  static_assert(IPT < 16, "four planes");
  uint32_t plane[4] = {0, 0, 0, 0};
#pragma unroll
  for (int j = 0; j < IPT; ++j) {
    const int a = A[j], d = min((int)D[j], kMaxDepth);
    uint32_t m = a <= d ? (2u << d) - (1u << a) : 0u;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const uint32_t carry = plane[k] & m;
      plane[k] ^= m;
      m = carry;
    }
  }
  const uint32_t any = plane[0] | plane[1] | plane[2] | plane[3];
#pragma unroll
  for (int wi = 0; wi < kLevelWords; ++wi) {
    c[wi] = 0;
    if (__ballot((any >> (2 * wi)) & 3u) != 0) {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        // bits 0 and 1 to bits 0 and 16
        const uint32_t two = (plane[k] >> (2 * wi)) & 3u;
        c[wi] += ((two * 0x8001u) & 0x10001u) << k;
      }
    }
  }
}

// The packed counters summed over the lanes up to each; the wave's totals go to wtot.
__device__ inline void wave_level_scan(uint32_t *wtot, const uint32_t c[kLevelWords],
                                       uint32_t inc[kLevelWords]) {
#pragma unroll
  for (int wi = 0; wi < kLevelWords; ++wi)
    inc[wi] = __ballot(c[wi]) != 0 ? wave_inclusive_scan(c[wi]) : 0u;
  if (lane_id() == 63) {
#pragma unroll
    for (int wi = 0; wi < kLevelWords; ++wi)
      wtot[threadIdx.x / 64 * kLevelWords + wi] = inc[wi];
  }
}

// Block-wide exclusive scan of the packed counters; the words that are 0 in the whole
// wave stay 0.  Leaves the waves' totals in wtot (published by the barrier).
__device__ inline void block_level_scan(uint32_t *wtot, uint32_t c[kLevelWords]) {
  const int wv = threadIdx.x / 64;
  uint32_t inc[kLevelWords];
  wave_level_scan(wtot, c, inc);
  __syncthreads();
#pragma unroll
  for (int wi = 0; wi < kLevelWords; ++wi) {
    if (__ballot(c[wi]) == 0) continue;
    uint32_t off = 0;
#pragma unroll
    for (int q = 0; q + 1 < kWaves; ++q) {
      const uint32_t v = wtot[q * kLevelWords + wi];
      off += (q < wv) ? v : 0u;
    }
    c[wi] = off + inc[wi] - c[wi];
  }
}

// The workgroup's cells at depth d, from the waves' totals.
__device__ __forceinline__ uint32_t block_level_total(const uint32_t *wtot, int d) {
  uint32_t t = 0;
#pragma unroll
  for (int q = 0; q < kWaves; ++q)
    t += (wtot[q * kLevelWords + (d >> 1)] >> ((d & 1) * 16)) & 0xffffu;
  return t;
}

__device__ __forceinline__ uint32_t unpack(const uint32_t w[kLevelWords], int d) {
  return (w[d >> 1] >> ((d & 1) * 16)) & 0xffffu;
}

// Tile t (of `tile` particles) of set b covers [t0, t1) inside the set's range [S, E).
struct TileRange {
  int b;
  int64_t S, E, t0, t1;
};

__device__ __forceinline__ TileRange tile_range(int64_t t, const int64_t *__restrict__ tile_start,
                                                const int32_t *__restrict__ tile_set,
                                                const int64_t *__restrict__ set_off,
                                                int tile) {
  TileRange r;
  r.b = tile_set[t];
  r.S = set_off[r.b];
  r.E = set_off[r.b + 1];
  r.t0 = r.S + (t - tile_start[r.b]) * (int64_t)tile;
  r.t1 = min(r.t0 + (int64_t)tile, r.E);
  return r;
}

#endif

}  // namespace tb
