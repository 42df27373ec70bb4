// tb_cells.hip -- leaves straight from the sorted keys (Sec. 2.3.1, Algorithm 1,
// Appendix A) and the level-ordered placement of every cell.
//
// Algorithm 1 walks the sorted keys once: the first particle k of a leaf gets
// the leaf depth D_k = max(minDepth(k-1, k), minDepth(k, k+n_leaf)) and the
// leaf absorbs the following particles that share its depth-D_k prefix.  Here
// the same leaves come out of a data-parallel form of that formula:
//
//   a_i = minDepth(i-1, i)            (0 for i = 0)
//   w_j = minDepth(j, j+n_leaf)       (for j + n_leaf < N, else 0)
//   D_i = min(21, max{ w_j : i - n_leaf <= j <= i })
//
// D_i is the depth of the leaf that holds particle i (a depth-d cell around i
// holds more than n_leaf particles exactly when some window [j, j+n_leaf]
// inside it contains i), and particle i is the first particle of the leaf
// exactly when a_i <= D_i -- where Algorithm 1 would start a new leaf.  For
// such a particle D_i equals the printed D_k.  The same particle is also the
// first particle of its ancestors at depths a_i .. D_i-1, which is how the
// bottom-up pass below knows, before any parent exists, how many cells each
// depth will hold and where each cell goes in the (depth, key) order.
//
// k_reorder    : particles in key order (the reorder step) and their keys; from
//                the keys of its tile plus an n_leaf halo, a_i and D_i of every
//                particle and the tile's per-depth cell counts;
// k_cell_scan  : per-depth prefix over the tiles of each set;
// k_set_scan_* : first cell of every set and depth (one set of few tiles: both in
//                k_cell_emit);
// k_cell_emit  : writes key, depth, first particle and first-child slot of
//                every cell, and count plus moments of every leaf.
// (With TB_SUBTREES the cells are written block by block instead:
// tb_blocks.hip.)
#include "tb_internal.h"
#include "tb_moments.h"
#include "tb_tiles.h"

namespace tb {


__host__ __device__ constexpr size_t round16(size_t x) { return (x + 15) & ~size_t(15); }

// Particles of the reorder's window: the tile, the n_leaf + 1 before and n_leaf after
// it, and `ext` more on either side.
__host__ __device__ constexpr int window_size(int tile, int nl, int ext) {
  return tile + 2 * nl + 1 + 2 * ext;
}
// A thread gathers IPT + 1 of the window's particles at once.  If that holds the window
// with the ends of its runs (n_leaf <= 95 for either tile) the reorder finishes the sort;
// larger windows get particles that the radix passes have sorted by all key bits
// (make_plan).
__host__ __device__ constexpr int window_ext(int nl) {
  return window_size(kCellTile, nl, kRunCap) <= (kCellIpt + 1) * kCellThreads ? kRunCap : 0;
}
static_assert((kCellIpt + 1) * kCellThreads - kCellTile ==
                  (kSmallIpt + 1) * kCellThreads - kSmallTile,
              "both tiles leave the same room beside them");
bool reorder_finishes(int nl) { return window_ext(nl) != 0; }

// Shared layout of the reorder pass (dynamic LDS, sized for the actual n_leaf).
struct WindowLds {
  uint64_t *raw;   // [window]        keys in the order the radix passes left, then the
                   //                 final one
  uint64_t *heads; // [window / 64]   where the window's runs start, a word of ones before
                   //                 and after them (if the reorder finishes the sort)
  uint64_t *keys;  // [T + 2 NL + 1]  the final keys of [t0 - NL - 1, t1 + NL)
  uint8_t *m;      // [T + NL]        w_j, then the sparse max table, j in [t0 - NL, t1)
  uint8_t *a;      // [T + NL]        a_i, i in [t0, t1 + NL)
  uint32_t *wtot;  // [kWaves][kLevelWords]
};

__host__ __device__ inline size_t window_keys_bytes(int nl, int tile) {
  return round16((size_t)window_size(tile, nl, window_ext(nl)) * 8);
}

// (rows of kCellThreads particles, kWaves words each)
__host__ __device__ inline size_t window_heads_bytes(int nl, int tile) {
  return window_ext(nl) ? round16((size_t)((tile / kCellThreads + 1) * kWaves + 2) * 8) : 0;
}

__host__ __device__ inline size_t window_lds_bytes(int nl, int tile) {
  return window_keys_bytes(nl, tile) + window_heads_bytes(nl, tile) + 2 * round16(tile + nl) +
         (size_t)kWaves * kLevelWords * 4;
}

__device__ inline WindowLds carve_window(unsigned char *base, int nl, int tile) {
  WindowLds s;
  s.raw = reinterpret_cast<uint64_t *>(base);
  s.keys = s.raw + window_ext(nl);
  base += window_keys_bytes(nl, tile);
  s.heads = reinterpret_cast<uint64_t *>(base);
  base += window_heads_bytes(nl, tile);
  s.m = base;
  base += round16(tile + nl);
  s.a = base;
  base += round16(tile + nl);
  s.wtot = reinterpret_cast<uint32_t *>(base);
  return s;
}

// Shared layout of the emit pass.
struct EmitLds {
  uint8_t *a;          // [T + NL]        a_i, i in [t0, t1 + NL)
  uint8_t *d;          // [T]             D_i, i in [t0, t1)
  uint32_t *wtot;      // [kWaves][kLevelWords]
  uint32_t *lvl;       // [kLevels]       first slot of the depth's cells of this tile, less
                       //                 the tile's cells at smaller depths
  uint16_t *off;       // [kLevels][kCellThreads] next cell per depth per thread
  float4 *rec;         // [T + NL]        sorted (x, y, z, m) of [t0, t1 + NL); stored once
                       //                 the cells are listed, over the dead `off` and `list`
  uint32_t *list;      // [T]             cells starting in the tile (k_cell_emit); beside
                       //                 `off`, and read into registers before `rec` is stored
  uint8_t *heads;      // [T / 8]         bit li: particle t0 + li starts a leaf
  uint32_t *nleaf;     // [1]
};

__host__ __device__ inline size_t emit_off_bytes() {
  return round16((size_t)kLevels * kCellThreads * 2);
}

__host__ __device__ inline size_t emit_union_bytes(int nl, int tile) {
  const size_t cells = emit_off_bytes() + (size_t)tile * 4;  // off, then list
  const size_t rec = (size_t)(tile + nl) * 16;
  return round16(cells > rec ? cells : rec);
}

__host__ __device__ inline size_t emit_lds_bytes(int nl, int tile) {
  return round16(tile + nl) + round16(tile) + round16((size_t)kWaves * kLevelWords * 4) +
         round16(kLevels * 4) + emit_union_bytes(nl, tile) + tile / 8 + 16;
}

__device__ inline EmitLds carve_emit(unsigned char *base, int nl, int tile) {
  EmitLds s;
  s.a = base;
  base += round16(tile + nl);
  s.d = base;
  base += round16(tile);
  s.wtot = reinterpret_cast<uint32_t *>(base);
  base += round16((size_t)kWaves * kLevelWords * 4);
  s.lvl = reinterpret_cast<uint32_t *>(base);
  base += round16(kLevels * 4);
  // the per-depth cursors and the list are dead once the cells are listed
  // (each thread keeps its entries in registers); the particle records
  // take their place for the moment phase
  s.off = reinterpret_cast<uint16_t *>(base);
  s.list = reinterpret_cast<uint32_t *>(base + emit_off_bytes());
  s.rec = reinterpret_cast<float4 *>(base);
  base += emit_union_bytes(nl, tile);
  s.heads = base;
  base += tile / 8;
  s.nleaf = reinterpret_cast<uint32_t *>(base);
  return s;
}

// From the key window in LDS (positions [t0 - nl - 1, t1 + nl), zero outside
// the set [S, E)): a_i and the windowed maximum, and (in A[], D[]) a_i and the
// leaf depth of this thread's IPT consecutive particles.  The set's first
// particle starts a root (a = 0) and windows never reach across the set's ends.
template <int IPT>
__device__ inline void depths_from_window(const WindowLds &s, int64_t S, int64_t E, int nl,
                                          int64_t t0, int64_t t1, uint8_t (&A)[IPT],
                                          uint8_t (&D)[IPT]) {
  constexpr int kMaxSpan =
      (IPT * kCellThreads + TB_MAX_NLEAF + kCellThreads - 1) / kCellThreads;
  const int T = (int)(t1 - t0);
  // a_i for i in [t0, t1 + nl)
  for (int i = threadIdx.x; i < T + nl; i += kCellThreads) {
    const int64_t g = t0 + i;
    uint8_t v = 0;
    if (g > S && g < E) v = (uint8_t)min_depth(s.keys[i + nl], s.keys[i + nl + 1]);
    s.a[i] = v;
  }
  // w_j for j in [t0 - nl, t1)
  for (int i = threadIdx.x; i < T + nl; i += kCellThreads) {
    const int64_t j = t0 - nl + i;
    uint8_t v = 0;
    if (j >= S && j + nl < E) v = (uint8_t)min_depth(s.keys[i + 1], s.keys[i + 1 + nl]);
    s.m[i] = v;
  }
  __syncthreads();
  // sparse table: after the loop m[x] = max(w[x .. x + 2^k - 1]) with 2^k <= nl + 1
  const int span = T + nl;
  int pk = 1;
  while (2 * pk <= nl + 1) {
    uint8_t tmp[kMaxSpan];
#pragma unroll
    for (int r = 0; r < kMaxSpan; ++r) {
      const int x = threadIdx.x + r * kCellThreads;
      uint8_t v = 0;
      if (x < span) {
        v = s.m[x];
        if (x + pk < span) v = max(v, s.m[x + pk]);
      }
      tmp[r] = v;
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kMaxSpan; ++r) {
      const int x = threadIdx.x + r * kCellThreads;
      if (x < span) s.m[x] = tmp[r];
    }
    __syncthreads();
    pk *= 2;
  }
  // window [i - nl, i] = [i - nl, i - nl + pk - 1] u [i - pk + 1, i]
#pragma unroll
  for (int j = 0; j < IPT; ++j) {
    const int li = threadIdx.x * IPT + j;  // particle t0 + li
    uint8_t d = 0, av = 23;
    if (li < T) {
      const int mx = max(s.m[li], s.m[li + nl + 1 - pk]);
      d = (uint8_t)min(mx, kMaxDepth);
      av = s.a[li];
    }
    A[j] = av;
    D[j] = d;
  }
}

// ---------------------------------------------------------------------------
// reorder pass (Sec. 2.3, step iii) with the leaf depths
// ---------------------------------------------------------------------------
// sorted[s] = packed[perm[s]]: the particles in key order, one 16-byte record
// each, and their keys recomputed from the gathered positions (the same FP64
// arithmetic as the key pass, so the keys are identical).  One workgroup per
// cell tile, so the whole tile shares one set and one root box.  The workgroup
// also gathers the n_leaf + 1 particles on either side of its tile (inside the
// set), which gives it the key window of the leaf-depth formula: it stores
// a_i | D_i << 8 for every particle of the tile and the tile's cell count per
// depth.  Every thread issues all of a batch's index loads, then all of its
// gathers, so the random reads overlap; they bound the pass (one 128-byte line a
// 16-byte record: 2^24 in random order, 2.1 GB of lines in 0.45 ms).  Also fills perm (if
// the sort has not) and the optional pos_sorted / mass_sorted / key_sorted outputs and
// checks the masses.
//
// The radix passes sort by the key bits from `skip` on, so a run of particles that
// agree in those arrives in input order.  A particle's place in its run follows from
// the run's other keys: those before it that are not larger and those after it that
// are smaller (which keeps equal keys in input order).  A window reaches kRunCap
// particles further than it needs, so every run of at most kRunCap particles that
// touches the needed part is whole, and a longer one looks longer.  A tile
// that meets a longer run writes nothing: it is listed, and so is the run if it starts
// in the tile; k_sort_runs sorts the listed runs, and a second launch does the listed
// tiles, where the particles of a longer run keep their places.  When the low bits were
// sorted too (*full) nothing is left to do.
struct ReorderArgs {
  const int32_t *order;  // the radix passes' indices
  const float4 *packed;
  int64_t n;
  int nl, skip, hilbert;
  const int64_t *tile_start;
  const int32_t *tile_set;
  const int64_t *set_off;
  int32_t nsets;
  const double *box;
  int64_t cell_tiles;
  const uint32_t *full, *oversize;
  uint32_t *n_runs, *n_run_tiles;
  int32_t *runs, *run_tiles;
  float4 *sorted;
  uint64_t *keys, *key_out;
  int32_t *perm;
  float *pos_sorted, *mass_sorted;
  uint16_t *ad;
  uint32_t *tile_cnt;
  int32_t *status_word;
};

// The window's runs, a bit a particle that does not agree with the one before it in the
// sorted bits (and every one outside the set), 64 particles a word, between two words
// of ones.
__device__ __forceinline__ uint64_t *run_heads(const WindowLds &s) { return s.heads + 1; }

// Places in the window of N particles, those at i0 + r * kCellThreads (i0 = threadIdx.x,
// so a wave holds 64 particles of one word): the number of the
// run's particles with smaller keys, or equal ones before it, after the run's start.
// Keys of a run differ below bit 31 only.  All of a thread's particles meet the d-th
// next of their runs (cyclically) in one step, as long as a run in the wave has more.
// Returns whether one of them is in a run longer than kRunCap (it keeps its place);
// *first: bit r if particle r is, and is the first of the run.
template <int N>
__device__ inline bool run_places(const WindowLds &s, int i0, int wn, const uint64_t (&key)[N],
                                  int (&place)[N], uint32_t *first) {
  const int lane = lane_id();
  const uint32_t *low = reinterpret_cast<const uint32_t *>(s.raw);  // low words at 2 i
  int end[N], len[N], most = 1;
  bool any = false;
  *first = 0;
#pragma unroll
  for (int r = 0; r < N; ++r) {
    const int i = i0 + r * kCellThreads, w = i / 64;
    end[r] = lane + 1;
    len[r] = 1;
    place[r] = i;
    if (i < wn) {
      const uint64_t *h = run_heads(s) + w;
      const uint64_t here = h[0], le = here & ((2ull << lane) - 1ull);
      const uint64_t gt = here & ~((2ull << lane) - 1ull);
      // relative to the word; beyond its neighbours the run is too long anyway
      const int start = le ? 63 - __clzll((long long)le)
                           : h[-1] ? -1 - __clzll((long long)h[-1]) : -64;
      end[r] = gt ? __ffsll((long long)gt) - 1 : h[1] ? 63 + __ffsll((long long)h[1]) : 128;
      len[r] = end[r] - start;
      if (len[r] > kRunCap) {
        any = true;
        if (start == lane) *first |= 1u << r;
        len[r] = 1;
      } else {
        place[r] += start - lane;
      }
      most = max(most, len[r]);
    }
  }
  for (int d = 1; __ballot(d < most) != 0; ++d) {
    uint32_t other[N];
#pragma unroll
    for (int r = 0; r < N; ++r) {
      const int j = lane + d, back = j >= end[r] ? len[r] : 0;
      // (past the run's particles: this one itself)
      const int at = d < len[r] ? i0 + r * kCellThreads + d - back : min(i0 + r * kCellThreads, wn - 1);
      other[r] = low[2 * at];
    }
#pragma unroll
    for (int r = 0; r < N; ++r) {
      const uint32_t mine = (uint32_t)key[r];
      const bool before = lane + d >= end[r];
      const bool smaller = other[r] < mine || (before && other[r] == mine);
      place[r] += d < len[r] && smaller ? 1 : 0;
    }
  }
  return any;
}

// FINISH: the window's records stay with the threads that gathered them until the
// particles' places are known.
template <bool FINISH, int IPT>
__device__ inline void reorder_tile(const ReorderArgs &g, const WindowLds &s, int64_t tile,
                                    bool again) {
  // a batch set over the caller's index bound: every particle gets the root key
  const bool flat = g.oversize && *g.oversize != 0u;
  const int nl = g.nl;
  const TileRange tr = tile_range(tile, g.tile_start, g.tile_set, g.set_off, IPT * kCellThreads);
  const int64_t t0 = tr.t0, t1 = tr.t1;
  const double lo0 = g.box[4 * tr.b + 0], lo1 = g.box[4 * tr.b + 1], lo2 = g.box[4 * tr.b + 2];
  const double scale = 2097152.0 / g.box[4 * tr.b + 3];
  const int T = (int)(t1 - t0);
  constexpr int kExt = FINISH ? kRunCap : 0;
  const int64_t ws = t0 - nl - 1 - kExt;  // window start (may be negative)
  const int wn = window_size(T, nl, kExt);
  constexpr int kBatch = IPT + 1;
  bool internal = false, bad = false;
  int32_t p[kBatch];
  float4 rec[kBatch];
  // particle r of a thread's batch to place i of the window
  auto put = [&](int r, int i, uint64_t key) {
    const int64_t q = ws + i;
    if (q < t0 || q >= t1) return;
    g.sorted[q] = rec[r];
    g.keys[q] = key;
    if (FINISH) g.perm[q] = p[r];  // (else the order is in perm)
    if (g.key_out) g.key_out[q] = key;
    bad |= !(rec[r].w > 0.0f && isfinite(rec[r].w));
    if (g.pos_sorted) {
      g.pos_sorted[3 * q + 0] = rec[r].x;
      g.pos_sorted[3 * q + 1] = rec[r].y;
      g.pos_sorted[3 * q + 2] = rec[r].z;
    }
    if (g.mass_sorted) g.mass_sorted[q] = rec[r].w;
  };
  // particles i0 + r * kCellThreads + threadIdx.x of the window
  auto gather = [&](int i0) {
#pragma unroll
    for (int r = 0; r < kBatch; ++r) {
      const int i = i0 + r * kCellThreads + threadIdx.x;
      const int64_t q = ws + i;
      const bool in = i < wn && q >= tr.S && q < tr.E;
      p[r] = g.order[in ? q : t0];
    }
#pragma unroll
    for (int r = 0; r < kBatch; ++r) {
      const int i = i0 + r * kCellThreads + threadIdx.x;
      const int64_t q = ws + i;
      const bool in = i < wn && q >= tr.S && q < tr.E;
      const bool ok = p[r] >= 0 && p[r] < g.n;
      internal |= in && !ok;
      rec[r] = g.packed[ok ? p[r] : 0];
    }
#pragma unroll
    for (int r = 0; r < kBatch; ++r) {
      const int i = i0 + r * kCellThreads + threadIdx.x;
      const int64_t q = ws + i;
      const bool in = i < wn && q >= tr.S && q < tr.E;
      const uint64_t key =
          !in ? 0ull
          : flat
              ? 1ull << 63
              : particle_key(rec[r].x, rec[r].y, rec[r].z, lo0, lo1, lo2, scale, g.hilbert != 0);
      if (i < wn) s.raw[i] = key;
      if (!FINISH && i < wn) put(r, i, key);
    }
  };
  if constexpr (!FINISH) {
    for (int i0 = 0; i0 < wn; i0 += kBatch * kCellThreads) gather(i0);
  } else {
    gather(0);
    __syncthreads();
    uint64_t key[kBatch];
    int place[kBatch];
#pragma unroll
    for (int r = 0; r < kBatch; ++r) {
      const int i = r * kCellThreads + threadIdx.x;
      key[r] = i < wn ? s.raw[i] : 0ull;
    }
    const bool whole = flat || *g.full != 0u;  // the order is final
    bool longer = false;
    if (!whole) {
#pragma unroll
      for (int r = 0; r < kBatch; ++r) {
        const int i = r * kCellThreads + threadIdx.x;
        bool head = true;
        if (i > 0 && i < wn) head = key[r] == 0ull || ((key[r] ^ s.raw[i - 1]) >> g.skip) != 0;
        const uint64_t m = __ballot(head);
        if (lane_id() == 0) run_heads(s)[i / 64] = m;
      }
      if (threadIdx.x == 0) run_heads(s)[-1] = run_heads(s)[kBatch * kWaves] = ~0ull;
      __syncthreads();
      uint32_t first;
      longer = run_places<kBatch>(s, threadIdx.x, wn, key, place, &first);
#pragma unroll
      for (int r = 0; r < kBatch; ++r) {
        const int64_t q = ws + r * kCellThreads + threadIdx.x;
        if (((first >> r) & 1u) && !again && q >= t0 && q < t1)
          g.runs[atomicAdd(g.n_runs, 1u)] = (int32_t)q;
      }
    } else {
#pragma unroll
      for (int r = 0; r < kBatch; ++r) place[r] = r * kCellThreads + threadIdx.x;
    }
    // (every thread has read the keys it looks at)
    const bool stop = __syncthreads_or(longer ? 1 : 0) != 0 && !again;
    if (stop) {
      if (threadIdx.x == 0) g.run_tiles[atomicAdd(g.n_run_tiles, 1u)] = (int32_t)tile;
      return;
    }
#pragma unroll
    for (int r = 0; r < kBatch; ++r) {
      if (r * kCellThreads + (int)threadIdx.x >= wn) continue;
      s.raw[place[r]] = key[r];
      put(r, place[r], key[r]);
    }
  }
  if (__ballot(bad) != 0 && lane_id() == 0) atomicOr(g.status_word, TB_STATUS_MASS);
  if (__ballot(internal) != 0 && lane_id() == 0) atomicOr(g.status_word, TB_STATUS_INTERNAL);
  __syncthreads();

  uint8_t A[IPT], D[IPT];
  depths_from_window(s, tr.S, tr.E, nl, t0, t1, A, D);
#pragma unroll
  for (int j = 0; j < IPT; ++j) {
    const int li = threadIdx.x * IPT + j;
    if (li < T) g.ad[t0 + li] = (uint16_t)(A[j] | (D[j] << 8));
  }
  uint32_t c[kLevelWords], inc[kLevelWords];
  thread_level_counts(A, D, c);
  wave_level_scan(s.wtot, c, inc);
  __syncthreads();
  const int d = threadIdx.x;
  if (d < kLevels) g.tile_cnt[d * g.cell_tiles + tile] = block_level_total(s.wtot, d);
}

template <bool FINISH, int IPT>
__global__ __launch_bounds__(kCellThreads, 4) void k_reorder(ReorderArgs g) {
  extern __shared__ __align__(16) unsigned char lds[];
  const int64_t tile = xcd_tile(blockIdx.x, gridDim.x);
  if (tile >= g.tile_start[g.nsets]) return;
  reorder_tile<FINISH, IPT>(g, carve_window(lds, g.nl, IPT * kCellThreads), tile, false);
}

// The tiles the first launch listed.
template <int IPT>
__global__ __launch_bounds__(kCellThreads) void k_reorder_again(ReorderArgs g) {
  extern __shared__ __align__(16) unsigned char lds[];
  const uint32_t n = *g.n_run_tiles;
  for (uint32_t q = blockIdx.x; q < n; q += gridDim.x) {
    reorder_tile<true, IPT>(g, carve_window(lds, g.nl, IPT * kCellThreads), g.run_tiles[q], true);
    __syncthreads();
  }
}

// Sorts each listed run of the radix passes' order by the key bits below `skip`, one
// workgroup a run.  The run lies in listed tiles only, whose sorted keys are not written
// yet, so keys0 and keys1 hold its (low bits << 32 | index) words.  Most runs are hardly
// longer than kRunCap: those below kRunFirst particles go by the ranks of their words in
// LDS.  A longer one (a clump too small for the sample to see: up to some 0.1 % of the
// particles) takes an LSD radix sort with 8-bit digits, kRunTile words at a time; a digit
// that all share takes no pass, and a run in order already (coincident particles) stays.
// What one CU gathers, ranks and scatters is what it costs, some 7 us a thousand particles:
// a clump of 80,000 in 2^26 uniform ones 588 us, of 12,000 in 2^24 92 us (1684 and 251 us
// with 256 words a step; 527 us with 1024 threads, 552 us with 16 words a thread); 1856
// short runs of 2^26 clustered particles 47 us.
constexpr int kRunThreads = 512, kRunItems = 8, kRunTile = kRunThreads * kRunItems;
constexpr int kRunFirst = 128;

__global__ __launch_bounds__(kRunThreads) void k_sort_runs(
    ReorderArgs g, int32_t *__restrict__ order, uint64_t *__restrict__ buf0,
    uint64_t *__restrict__ buf1) {
  constexpr int kDigits = 4, kRunWaves = kRunThreads / 64, kEdges = kRunItems * kRunWaves;
  static_assert(kRunThreads >= 256, "a thread for every digit");
  __shared__ uint32_t s_hist[kDigits][256];  // counts, then where each digit's words go
  __shared__ uint32_t s_wave[kRunWaves][256];
  __shared__ uint64_t s_first[kRunFirst];
  __shared__ uint32_t s_edge[kEdges + 1];  // low bits before each wave's first word
  __shared__ uint32_t s_w[4];
  __shared__ uint64_t s_pre;
  __shared__ int s_set, s_len;
  const uint32_t n_runs = *g.n_runs;
  const int t = threadIdx.x, wv = t / 64, lane = lane_id();
  const int digits = (g.skip + 7) / 8;
  for (uint32_t run = blockIdx.x; run < n_runs; run += gridDim.x) {
    const int64_t s = g.runs[run];
    if (t == 0) {
      s_set = upper_index(g.set_off, g.nsets + 1, s);
      s_len = 0;
    }
    for (int i = t; i < kDigits * 256; i += kRunThreads) (&s_hist[0][0])[i] = 0;
    __syncthreads();
    const int b = s_set;
    const int64_t E = g.set_off[b + 1];
    const double lo0 = g.box[4 * b + 0], lo1 = g.box[4 * b + 1], lo2 = g.box[4 * b + 2];
    const double scale = 2097152.0 / g.box[4 * b + 3];
    // the key of the particle with index idx
    auto key_of = [&](int32_t idx) {
      const float4 r = g.packed[idx >= 0 && idx < g.n ? idx : 0];
      return particle_key(r.x, r.y, r.z, lo0, lo1, lo2, scale, g.hilbert != 0);
    };
    const uint64_t low_mask = (1ull << g.skip) - 1;
    uint64_t key = 0, word = ~0ull;
    int32_t idx = 0;
    if (t < kRunFirst && s + t < E) {
      idx = order[s + t];
      key = key_of(idx);
    }
    if (t == 0) s_pre = key >> g.skip;
    __syncthreads();
    const uint64_t pre = s_pre;
    const bool in = t < kRunFirst && s + t < E && (key >> g.skip) == pre;
    if (in) word = (key & low_mask) << 32 | (uint32_t)idx;
    if (t < kRunFirst) s_first[t] = word;
    // a run is contiguous: its members are the first of what was looked at
    const int members = __syncthreads_count(in ? 1 : 0);
    if (members < kRunFirst) {
      if (in) {
        int rank = 0;
        for (int j = 0; j < members; ++j) rank += s_first[j] < word ? 1 : 0;
        order[s + rank] = idx;
      }
      __syncthreads();
      continue;
    }
    auto count = [&](uint32_t low) {
      for (int k = 0; k < digits; ++k) atomicAdd(&s_hist[k][(low >> (8 * k)) & 255u], 1u);
    };
    bool rising = true;
    if (in) {
      buf0[s + t] = word;
      count((uint32_t)(word >> 32));
      rising = t == 0 || (s_first[t - 1] >> 32) <= (word >> 32);
      if (t == kRunFirst - 1) s_edge[kEdges] = (uint32_t)(word >> 32);
    }
    // the rest of the run, up to the first particle past it
    for (int64_t c0 = s + kRunFirst;; c0 += kRunTile) {
      int32_t id[kRunItems];
      uint32_t low[kRunItems];
      bool has[kRunItems];
      int mine = 0;
#pragma unroll
      for (int r = 0; r < kRunItems; ++r) {
        const int64_t q = c0 + r * kRunThreads + t;
        id[r] = q < E ? order[q] : -1;
      }
#pragma unroll
      for (int r = 0; r < kRunItems; ++r) {
        const int64_t q = c0 + r * kRunThreads + t;
        const uint64_t k = key_of(id[r]);
        has[r] = q < E && (k >> g.skip) == pre;
        low[r] = (uint32_t)(k & low_mask);
      }
      __syncthreads();  // the edge before this step is written
      if (t == 0) s_edge[0] = s_edge[kEdges];
      __syncthreads();
#pragma unroll
      for (int r = 0; r < kRunItems; ++r) {
        if (has[r]) {
          buf0[c0 + r * kRunThreads + t] = (uint64_t)low[r] << 32 | (uint32_t)id[r];
          count(low[r]);
          ++mine;
        }
        const uint32_t before = __shfl_up(low[r], 1, 64);
        rising &= !has[r] || lane == 0 || before <= low[r];
        if (lane == 63) s_edge[1 + r * kRunWaves + wv] = low[r];
      }
      const uint32_t sum = wave_inclusive_scan((uint32_t)mine);
      if (lane == 63) atomicAdd(&s_len, (int)sum);
      const bool whole = __syncthreads_and(mine == kRunItems ? 1 : 0) != 0;
#pragma unroll
      for (int r = 0; r < kRunItems; ++r)
        rising &= !has[r] || lane != 0 || s_edge[r * kRunWaves + wv] <= low[r];
      if (!whole) break;
    }
    const int len = kRunFirst + s_len;
    if (__syncthreads_and(rising ? 1 : 0)) continue;
    uint64_t *src = buf0 + s, *dst = buf1 + s;
    for (int k = 0; k < digits; ++k) {
      const int sh = 32 + 8 * k;
      if (s_hist[k][(src[0] >> sh) & 255u] == (uint32_t)len) continue;  // the same for all
      {
        const uint32_t v = t < 256 ? s_hist[k][t] : 0u, inc = wave_inclusive_scan(v);
        if (lane == 63 && wv < 4) s_w[wv] = inc;
        __syncthreads();
        uint32_t off = inc - v;
        for (int q = 0; q < wv && q < 4; ++q) off += s_w[q];
        if (t < 256) s_hist[k][t] = off;
      }
      // a tile at a time, in order: a wave's words lie together, ranks by ballots within it
      for (int c0 = 0; c0 < len; c0 += kRunTile) {
        uint64_t w[kRunItems];
        uint32_t rk[kRunItems];
        const int i0 = c0 + wv * 64 * kRunItems + lane;
#pragma unroll
        for (int r = 0; r < kRunItems; ++r) w[r] = src[min(i0 + r * 64, len - 1)];
        for (int i = t; i < kRunWaves * 256; i += kRunThreads) (&s_wave[0][0])[i] = 0;
        __syncthreads();
#pragma unroll
        for (int r = 0; r < kRunItems; ++r) {
          const bool have = i0 + r * 64 < len;
          const uint32_t d = (uint32_t)(w[r] >> sh) & 255u;
          uint64_t peers = __ballot(have);
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            const bool bit = (d >> i) & 1u;
            const uint64_t m = __ballot(bit);
            peers &= bit ? m : ~m;
          }
          const uint32_t before = (uint32_t)__popcll(peers & lanemask_lt());
          const uint32_t was = s_wave[wv][d];
          rk[r] = was + before;
          if (have && before == 0) s_wave[wv][d] = was + (uint32_t)__popcll(peers);
        }
        __syncthreads();
        if (t < 256) {
          uint32_t at = s_hist[k][t];
#pragma unroll
          for (int q = 0; q < kRunWaves; ++q) {
            const uint32_t c = s_wave[q][t];
            s_wave[q][t] = at;
            at += c;
          }
          s_hist[k][t] = at;
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < kRunItems; ++r)
          if (i0 + r * 64 < len) dst[s_wave[wv][(w[r] >> sh) & 255u] + rk[r]] = w[r];
        __syncthreads();  // s_wave is read out
      }
      uint64_t *x = src;
      src = dst;
      dst = x;
    }
    for (int i = t; i < len; i += kRunThreads) order[s + i] = (int32_t)(uint32_t)src[i];
    __syncthreads();
  }
}

// Exclusive prefix of the per-tile counts over the earlier tiles of the same
// set, one workgroup per (depth, set); the set's total per depth goes to
// set_tot[b][d].  A single set uses 1024-thread workgroups (8192 tiles, i.e.
// 2^24 particles, per round), batches 256-thread ones (their sets are small).
constexpr int kScanItems = 8;

template <int THREADS>
__global__ __launch_bounds__(THREADS) void k_cell_scan(
    const uint32_t *__restrict__ tile_cnt, int64_t cell_tiles,
    const int64_t *__restrict__ tile_start, int32_t nsets, uint32_t *__restrict__ excl,
    uint32_t *__restrict__ set_tot) {
  __shared__ uint32_t s_w[THREADS / 64];
  const int d = blockIdx.x;
  const uint32_t *row = tile_cnt + d * cell_tiles;
  uint32_t *out = excl + d * cell_tiles;
  const int wv = threadIdx.x / 64;
  for (int b = blockIdx.y; b < nsets; b += gridDim.y) {
    const int64_t ts = tile_start[b], te = tile_start[b + 1];
    uint32_t carry = 0;
    for (int64_t c0 = ts; c0 < te; c0 += (int64_t)THREADS * kScanItems) {
      const int64_t q = c0 + (int64_t)threadIdx.x * kScanItems;
      uint32_t v[kScanItems], sum = 0;
#pragma unroll
      for (int r = 0; r < kScanItems; ++r) v[r] = (q + r < te) ? row[q + r] : 0u;
#pragma unroll
      for (int r = 0; r < kScanItems; ++r) sum += v[r];
      const uint32_t inc = wave_inclusive_scan(sum);
      if (lane_id() == 63) s_w[wv] = inc;
      __syncthreads();
      uint32_t off = 0, tot = 0;
#pragma unroll
      for (int k = 0; k < THREADS / 64; ++k) {
        const uint32_t t = s_w[k];
        off += (k < wv) ? t : 0u;
        tot += t;
      }
      __syncthreads();
      uint32_t run = carry + off + inc - sum;
#pragma unroll
      for (int r = 0; r < kScanItems; ++r) {
        if (q + r < te) out[q + r] = run;
        run += v[r];
      }
      carry += tot;
    }
    if (threadIdx.x == 0) set_tot[b * kLevels + d] = carry;
  }
}

// Rows of the set scan: 0 = cells per set; r = 1..21 = parent-pass chunks at
// depth r - 1 (children at depth r).
__device__ inline void set_rows(const uint32_t *__restrict__ set_tot, int32_t nsets, int b,
                                uint32_t t[kLevels], uint32_t v[kLevels]) {
#pragma unroll
  for (int d = 0; d < kLevels; ++d) t[d] = (b < nsets) ? set_tot[b * kLevels + d] : 0u;
  v[0] = 0;
#pragma unroll
  for (int d = 0; d < kLevels; ++d) v[0] += t[d];
#pragma unroll
  for (int r = 1; r < kLevels; ++r) v[r] = (t[r] + kParentChunk - 1) / kParentChunk;
}

// Sets [b0, b0 + THREADS), one per thread, every row at once, given in s_carry
// the sums of every row over the sets before b0: writes the first cell of every
// set and of every depth of every set (level_offset [B][23], cell_offsets), the
// parent-pass chunk tables and the boxes used, and leaves in s_w the block's
// per-wave row sums.
template <int THREADS>
__device__ inline void set_scan_block(
    int b0, const uint32_t *__restrict__ set_tot, int32_t nsets, int64_t *__restrict__ set_cells,
    int64_t *__restrict__ lvl_off, int64_t *__restrict__ level_offset,
    int64_t *__restrict__ cell_offsets, int64_t *__restrict__ par_start,
    const double *__restrict__ box, double *__restrict__ box_out,
    uint32_t (*s_w)[THREADS / 64], const int64_t *s_carry) {
  const int wv = threadIdx.x / 64;
  const int b = b0 + threadIdx.x;
  uint32_t t[kLevels], v[kLevels], inc[kLevels];
  set_rows(set_tot, nsets, b, t, v);
#pragma unroll
  for (int r = 0; r < kLevels; ++r) inc[r] = wave_inclusive_scan(v[r]);
  if (lane_id() == 63) {
#pragma unroll
    for (int r = 0; r < kLevels; ++r) s_w[r][wv] = inc[r];
  }
  __syncthreads();
  int64_t off[kLevels];
#pragma unroll
  for (int r = 0; r < kLevels; ++r) {
    int64_t o = s_carry[r];
    for (int q = 0; q < wv; ++q) o += s_w[r][q];
    off[r] = o + (int64_t)(inc[r] - v[r]);
  }
  if (b < nsets) {
    set_cells[b] = off[0];
    if (cell_offsets) cell_offsets[b] = off[0];
    int64_t run = off[0];
#pragma unroll
    for (int d = 0; d < kLevels; ++d) {
      lvl_off[b * (kLevels + 1) + d] = run;
      level_offset[b * (kLevels + 1) + d] = run;
      run += t[d];
    }
    lvl_off[b * (kLevels + 1) + kLevels] = run;
    level_offset[b * (kLevels + 1) + kLevels] = run;
    if (box_out)
      for (int k = 0; k < 4; ++k) box_out[4 * b + k] = box[4 * b + k];
#pragma unroll
    for (int r = 1; r < kLevels; ++r) par_start[(r - 1) * (nsets + 1) + b] = off[r];
  }
}

// The totals over all sets: set_cells[B], cell_offsets[B], n_cells and the last
// entry of every parent-pass chunk table (thread r < kLevels writes row r).
__device__ inline void set_scan_totals(int r, int64_t total, int32_t nsets,
                                       int64_t *__restrict__ set_cells,
                                       int64_t *__restrict__ cell_offsets,
                                       int64_t *__restrict__ n_cells,
                                       int64_t *__restrict__ par_start) {
  if (r == 0) {
    set_cells[nsets] = total;
    if (cell_offsets) cell_offsets[nsets] = total;
    *n_cells = total;
  } else {
    par_start[(r - 1) * (nsets + 1) + nsets] = total;
  }
}

// Up to 64 sets: one wave does the whole scan.
__global__ __launch_bounds__(64) void k_set_scan_wave(
    const uint32_t *__restrict__ set_tot, int32_t nsets, int64_t *__restrict__ set_cells,
    int64_t *__restrict__ lvl_off, int64_t *__restrict__ level_offset,
    int64_t *__restrict__ cell_offsets, int64_t *__restrict__ n_cells,
    int64_t *__restrict__ par_start, const double *__restrict__ box,
    double *__restrict__ box_out) {
  __shared__ uint32_t s_w[kLevels][1];
  __shared__ int64_t s_carry[kLevels];
  if (threadIdx.x < kLevels) s_carry[threadIdx.x] = 0;
  __syncthreads();
  set_scan_block<64>(0, set_tot, nsets, set_cells, lvl_off, level_offset, cell_offsets,
                     par_start, box, box_out, s_w, s_carry);
  __syncthreads();
  if (threadIdx.x < kLevels)
    set_scan_totals(threadIdx.x, (int64_t)s_w[threadIdx.x][0], nsets, set_cells, cell_offsets,
                    n_cells, par_start);
}

// More sets: THREADS sets per workgroup over G workgroups, in two launches.
// k_set_sums writes the row sums of each workgroup's sets, wg_sum[g][r];
// k_set_scan_wg adds the sums of the earlier workgroups to its own block scan.
// A set's row is read and written by one thread, some 70 scattered words, so a few
// sets are spread over more CUs: 64 a workgroup up to kFewSets (300 sets: 9.2 us in 2
// workgroups, 7.0 us in 5), but 256 beyond, where each workgroup's sum over the
// earlier ones would be long.
template <int THREADS>
__global__ __launch_bounds__(THREADS) void k_set_sums(
    const uint32_t *__restrict__ set_tot, int32_t nsets, int64_t *__restrict__ wg_sum) {
  constexpr int W = THREADS / 64;
  __shared__ uint32_t s_w[kLevels][W];
  uint32_t t[kLevels], v[kLevels];
  set_rows(set_tot, nsets, blockIdx.x * THREADS + threadIdx.x, t, v);
#pragma unroll
  for (int r = 0; r < kLevels; ++r) {
    const uint32_t inc = wave_inclusive_scan(v[r]);
    if (lane_id() == 63) s_w[r][threadIdx.x / 64] = inc;
  }
  __syncthreads();
  if (threadIdx.x < kLevels) {
    int64_t tot = 0;
    for (int q = 0; q < W; ++q) tot += s_w[threadIdx.x][q];
    wg_sum[blockIdx.x * kLevels + threadIdx.x] = tot;
  }
}

template <int THREADS>
__global__ __launch_bounds__(THREADS) void k_set_scan_wg(
    const uint32_t *__restrict__ set_tot, int32_t nsets, const int64_t *__restrict__ wg_sum,
    int64_t *__restrict__ set_cells, int64_t *__restrict__ lvl_off,
    int64_t *__restrict__ level_offset, int64_t *__restrict__ cell_offsets,
    int64_t *__restrict__ n_cells, int64_t *__restrict__ par_start,
    const double *__restrict__ box, double *__restrict__ box_out) {
  constexpr int W = THREADS / 64;
  __shared__ uint32_t s_w[kLevels][W];
  __shared__ int64_t s_carry[kLevels];
  if (threadIdx.x < kLevels) {
    int64_t c = 0;
    for (int g = 0; g < (int)blockIdx.x; ++g) c += wg_sum[g * kLevels + threadIdx.x];
    s_carry[threadIdx.x] = c;
  }
  __syncthreads();
  set_scan_block<THREADS>(blockIdx.x * THREADS, set_tot, nsets, set_cells,
                                  lvl_off, level_offset, cell_offsets, par_start, box, box_out,
                                  s_w, s_carry);
  __syncthreads();
  if (blockIdx.x + 1 == gridDim.x && threadIdx.x < kLevels) {
    int64_t tot = s_carry[threadIdx.x];
    for (int q = 0; q < W; ++q) tot += s_w[threadIdx.x][q];
    set_scan_totals(threadIdx.x, tot, nsets, set_cells, cell_offsets, n_cells, par_start);
  }
}

// ---------------------------------------------------------------------------
// leaf moments
// ---------------------------------------------------------------------------

// End (exclusive) of the leaf that starts at particle i with depth dl, from
// the a_i of the particles after it (a: [t0, t1 + nl) relative to t0).
__device__ inline int64_t leaf_end(const uint8_t *a, const uint64_t *__restrict__ keys, int64_t n,
                                   int nl, int64_t t0, int64_t i, int dl) {
  // n is the end of the particle's set
  const int64_t lim = min(n, i + nl + 1);
  for (int64_t j = i + 1; j < lim; ++j)
    if (a[j - t0] <= dl) return j;
  if (lim == n) return n;
  // only a depth-21 leaf of identical keys can be longer than n_leaf
  const uint64_t k = keys[i];
  int64_t lo = i + nl + 1, hi = n;  // first index in [lo, hi) whose key differs
  while (lo < hi) {
    const int64_t mid = lo + (hi - lo) / 2;
    if (keys[mid] == k)
      lo = mid + 1;
    else
      hi = mid;
  }
  return lo;
}

// The same leaf end from the tile's head mask: a leaf ends where the next leaf
// starts (a particle inside the leaf shares the leaf's prefix with its
// predecessor, so it starts no cell; the first particle past the leaf differs
// from its predecessor at depth <= the leaf depth and starts its own leaf).
// Only a leaf reaching past the tile falls back to the halo scan.
__device__ inline int64_t leaf_end_fast(const EmitLds &s, const uint64_t *__restrict__ keys,
                                        int64_t n, int nl, int64_t t0, int T, int li, int dl) {
  const uint64_t *hw = reinterpret_cast<const uint64_t *>(s.heads);
  const int nw = (T + 63) >> 6;
  int w = li >> 6;
  const int b = li & 63;
  uint64_t bits = b == 63 ? 0ull : (hw[w] >> (b + 1)) << (b + 1);
  while (bits == 0 && ++w < nw) bits = hw[w];
  if (bits != 0) {
    const int p = (w << 6) + __ffsll((long long)bits) - 1;
    if (p < T) return t0 + p;
  }
  return leaf_end(s.a, keys, n, nl, t0, t0 + li, dl);
}

// ---------------------------------------------------------------------------
// prefixes of one set with few tiles
// ---------------------------------------------------------------------------
// The scans' outputs, and the counts they are taken from.
struct SetScan {
  const uint32_t *tile_cnt;  // null: k_cell_scan and k_set_scan_* have run
  uint32_t *excl;
  int64_t *set_cells, *lvl_off, *level_offset, *cell_offsets, *n_cells, *par_start;
  const double *box;
  double *box_out;
};

// With one set of at most kFewTiles tiles the emit pass takes the prefixes over the tile
// counts itself, every workgroup its own (22 depths of at most 1 KB each, all loads in
// flight at once), instead of waiting for two launches that do little: 2^16 particles
// 119.5 -> 114.1 us (7 us of launches for 2 us in the emit pass).  The first tile's
// workgroup writes what the set scan would.
constexpr int kFewTiles = 256;
bool few_tiles(const Plan &p) {
  return p.nsets == 1 && p.cell_tiles <= kFewTiles && !(p.flags & TB_SUBTREES);
}

// A wave's share: its depths' cells of the earlier tiles (s_before[d]) and of all tiles
// (s_all[d]).
__device__ inline void tile_prefixes(const SetScan &g, int64_t tile, int tiles,
                                     int64_t cell_tiles, uint32_t *s_before, uint32_t *s_all) {
  constexpr int kDepths = (kLevels + kWaves - 1) / kWaves, kLoads = kFewTiles / 64;
  const int wv = threadIdx.x / 64, lane = lane_id();
  uint32_t v[kDepths][kLoads];
#pragma unroll
  for (int r = 0; r < kDepths; ++r) {
    const int d = wv + r * kWaves;
#pragma unroll
    for (int u = 0; u < kLoads; ++u) {
      const int q = lane + u * 64;
      v[r][u] = d < kLevels && q < tiles ? g.tile_cnt[d * cell_tiles + q] : 0u;
    }
  }
#pragma unroll
  for (int r = 0; r < kDepths; ++r) {
    const int d = wv + r * kWaves;
    uint32_t before = 0, all = 0;
#pragma unroll
    for (int u = 0; u < kLoads; ++u) {
      all += v[r][u];
      before += lane + u * 64 < tile ? v[r][u] : 0u;
    }
    before = wave_inclusive_scan(before);
    all = wave_inclusive_scan(all);
    if (lane == 63 && d < kLevels) {
      s_before[d] = before;
      s_all[d] = all;
    }
  }
}

// The first wave: lane d gets the tile's first slot at depth d and writes its outputs.
__device__ inline uint32_t set_prefix(const SetScan &g, int64_t tile, int64_t cell_tiles,
                                      const uint32_t *s_before, const uint32_t *s_all) {
  const int d = lane_id();
  const uint32_t before = d < kLevels ? s_before[d] : 0u, all = d < kLevels ? s_all[d] : 0u;
  const uint32_t upto = wave_inclusive_scan(all), first = upto - all;
  if (d < kLevels) g.excl[d * cell_tiles + tile] = before;
  if (tile == 0) {
    if (d <= kLevels) {  // (lane kLevels: the total)
      g.lvl_off[d] = first;
      g.level_offset[d] = first;
    }
    if (d == kLevels) {
      g.set_cells[0] = 0;
      g.set_cells[1] = first;
      *g.n_cells = first;
      if (g.cell_offsets) {
        g.cell_offsets[0] = 0;
        g.cell_offsets[1] = first;
      }
    }
    if (d > 0 && d < kLevels) {
      g.par_start[2 * (d - 1)] = 0;
      g.par_start[2 * (d - 1) + 1] = (all + kParentChunk - 1) / kParentChunk;
    }
    if (d < 4 && g.box_out) g.box_out[d] = g.box[d];
  }
  return first + before;
}

// ---------------------------------------------------------------------------
// emit pass
// ---------------------------------------------------------------------------
// One workgroup per cell tile: a_i and D_i (from the reorder pass) give every
// cell whose first particle lies in the tile; the per-depth prefix places it.
//
// The tile's cells are listed in LDS in the order of the output (depth, then place), and
// then written one a lane: neighbouring lanes write neighbouring cells.  Each thread
// writing the cells of its own particles sent 1.7 times the write requests, in three times
// the store instructions, and kept the address units busy 3/4 of the time: 2^26 clustered
// particles 1570 us, 1211 us from the list (4.5 GB at 3.7 TB/s); 2^24 255 and 232 us.  A
// list entry is local first particle |
// depth << 11 | (internal cells) (first child's place in the list + 2^15) << 16.  A tile
// with more cells than particles (n_leaf of 1, or coincident pairs) has no room for the
// list: there each thread writes its cells as it finds them, and lists the leaves as
// local first particle | depth << 11 | place among the tile's cells << 16.
template <bool MIXED, int IPT>
__global__ __launch_bounds__(kCellThreads) void k_cell_emit(
    const uint64_t *__restrict__ keys, const uint16_t *__restrict__ ad, int nl,
    const uint32_t *__restrict__ excl, int64_t cell_tiles, const int64_t *__restrict__ tile_start,
    const int32_t *__restrict__ tile_set, const int64_t *__restrict__ set_off, int32_t nsets,
    const int64_t *__restrict__ lvl_off, const double *__restrict__ box,
    const float4 *__restrict__ sorted, uint64_t *__restrict__ cell_key,
    uint8_t *__restrict__ cell_level, int32_t *__restrict__ cell_first,
    int32_t *__restrict__ cell_count, int32_t *__restrict__ child_ptr, void *__restrict__ com_v,
    void *__restrict__ quad_v, float *__restrict__ m_lo, int32_t *__restrict__ head_parent,
    int64_t c_max, int hilbert, int32_t *__restrict__ status_word, SetScan scan) {
  extern __shared__ __align__(16) unsigned char lds[];
  constexpr int kTile = IPT * kCellThreads;
  const EmitLds s = carve_emit(lds, nl, kTile);
  const int64_t tile = xcd_tile(blockIdx.x, gridDim.x);
  if (tile >= tile_start[nsets]) return;
  const TileRange tr = tile_range(tile, tile_start, tile_set, set_off, kTile);
  const int64_t t0 = tr.t0, t1 = tr.t1, n = tr.E;  // n: end of this tile's set
  const int T = (int)(t1 - t0);
  // the structure of cell ci at depth d, from its first particle i and that one's key;
  // fc: its first child, or -1
  auto put_cell = [&](uint32_t ci, uint64_t key, int d, int64_t i, int32_t fc) {
    cell_key[ci] = key >> (63 - 3 * d);
    cell_level[ci] = (uint8_t)d;
    cell_first[ci] = (int32_t)i;
    reinterpret_cast<int2 *>(child_ptr)[ci] = make_int2(fc, 0);
    if (head_parent && fc >= 0 && (int64_t)fc < c_max) head_parent[fc] = (int32_t)ci;
  };

  // per-depth base of this tile: the set's first cell of the depth plus the
  // cells of the set's earlier tiles
  uint32_t base = 0;
  uint32_t *s_before = reinterpret_cast<uint32_t *>(s.off);  // not used yet
  uint32_t *s_all = s_before + kLevels;
  if (scan.tile_cnt) {
    tile_prefixes(scan, tile, (int)tile_start[nsets], cell_tiles, s_before, s_all);
  } else if (threadIdx.x < kLevels) {
    const int d = threadIdx.x;
    base = (uint32_t)(lvl_off[tr.b * (kLevels + 1) + d] + excl[d * cell_tiles + tile]);
  }
  if (threadIdx.x == 0) *s.nleaf = 0;
  // the (a, D) of the tile's particles and the n_leaf halo into LDS, in one
  // batch of loads
  const int span = (int)(min(t1 + (int64_t)nl, n) - t0);
  constexpr int kRecBatch = IPT + 1;  // covers span for n_leaf <= 256
  for (int x0 = 0; x0 < span; x0 += kRecBatch * kCellThreads) {
    uint16_t v[kRecBatch];
#pragma unroll
    for (int u = 0; u < kRecBatch; ++u) {
      const int x = x0 + u * kCellThreads + threadIdx.x;
      v[u] = ad[t0 + (x < span ? x : span - 1)];
    }
#pragma unroll
    for (int u = 0; u < kRecBatch; ++u) {
      const int x = x0 + u * kCellThreads + threadIdx.x;
      if (x < span) {
        s.a[x] = (uint8_t)(v[u] & 0xff);
        if (x < T) s.d[x] = (uint8_t)(v[u] >> 8);
      }
    }
  }
  __syncthreads();
  // (before the next barrier, after which s.off is written)
  if (scan.tile_cnt && threadIdx.x < 64) base = set_prefix(scan, tile, cell_tiles, s_before, s_all);
  uint8_t A[IPT], D[IPT];
#pragma unroll
  for (int j = 0; j < IPT; ++j) {
    const int li = threadIdx.x * IPT + j;
    A[j] = li < T ? s.a[li] : 23;  // 23: starts no cell
    D[j] = li < T ? s.d[li] : 0;
  }
  {
    // the head mask: bit li is particle t0 + li (none past the tile end), IPT bits a
    // thread, a byte from 8 / IPT neighbours
    static_assert(IPT == 8 || IPT == 2, "threads make up whole bytes of the head mask");
    uint32_t hb = 0;
#pragma unroll
    for (int j = 0; j < IPT; ++j) hb |= (A[j] <= D[j] ? 1u : 0u) << j;
    constexpr int kShare = 8 / IPT;
    if constexpr (kShare > 1) {
      hb <<= (threadIdx.x % kShare) * IPT;
#pragma unroll
      for (int o = 1; o < kShare; o <<= 1) hb |= __shfl_xor(hb, o, 64);
    }
    if (threadIdx.x % kShare == 0) s.heads[threadIdx.x / kShare] = (uint8_t)hb;
  }
  uint32_t c[kLevelWords];
  thread_level_counts(A, D, c);
  block_level_scan(s.wtot, c);  // its barrier also publishes s.heads
  // the tile's cells at smaller depths (lane d: before depth d)
  const uint32_t cnt = lane_id() < kLevels ? block_level_total(s.wtot, lane_id()) : 0u;
  const uint32_t upto = wave_inclusive_scan(cnt);
  const int ncells = __builtin_amdgcn_readlane((int)upto, 63);
  const bool listed = ncells <= kTile;
  if (threadIdx.x < kLevels) s.lvl[threadIdx.x] = base - (upto - cnt);
#pragma unroll
  for (int d = 0; d < kLevels; ++d)
    s.off[d * kCellThreads + threadIdx.x] =
        (uint16_t)(unpack(c, d) + (uint32_t)__builtin_amdgcn_readlane((int)(upto - cnt), d));

  bool internal = false;
  int nlist = ncells;
  if (listed) {
#pragma unroll
    for (int j = 0; j < IPT; ++j) {
      const int a = A[j], dl = D[j];
      if (a > dl) continue;
      const uint32_t li = threadIdx.x * IPT + j;
      uint32_t x = s.off[a * kCellThreads + threadIdx.x];
      for (int d = a; d < dl; ++d) {
        s.off[d * kCellThreads + threadIdx.x] = (uint16_t)(x + 1);
        // first child: this particle's cell one depth down
        const uint32_t xc = s.off[(d + 1) * kCellThreads + threadIdx.x];
        if (x < (uint32_t)kTile) s.list[x] = li | ((uint32_t)d << 11) | ((xc | 0x8000u) << 16);
        x = xc;
      }
      s.off[dl * kCellThreads + threadIdx.x] = (uint16_t)(x + 1);
      if (x < (uint32_t)kTile) s.list[x] = li | ((uint32_t)dl << 11);
    }
  } else {
    // this thread's leaves go to a contiguous run of the list
    uint64_t kk[IPT];
    uint32_t my_leaves = 0;
#pragma unroll
    for (int j = 0; j < IPT; ++j) {
      const int li = threadIdx.x * IPT + j;
      kk[j] = keys[t0 + (li < T ? li : T - 1)];
      my_leaves += (A[j] <= D[j]) ? 1u : 0u;
    }
    const uint32_t inc = wave_inclusive_scan(my_leaves);
    uint32_t wave_base = 0;
    if (lane_id() == 63) wave_base = atomicAdd(s.nleaf, inc);
    wave_base = __shfl(wave_base, 63, 64);
    uint32_t leaf_slot = wave_base + inc - my_leaves;
    __syncthreads();  // s.lvl
#pragma unroll
    for (int j = 0; j < IPT; ++j) {
      const int a = A[j], dl = D[j];
      if (a > dl) continue;
      const int li = threadIdx.x * IPT + j;
      for (int d = a; d <= dl; ++d) {
        const uint32_t x = s.off[d * kCellThreads + threadIdx.x];
        s.off[d * kCellThreads + threadIdx.x] = (uint16_t)(x + 1);
        const uint32_t ci = s.lvl[d] + x;
        if ((int64_t)ci >= c_max) {  // cannot happen with consistent counts
          internal = true;
          continue;
        }
        int32_t fc = -1;
        if (d < dl) {
          fc = (int32_t)(s.lvl[d + 1] + s.off[(d + 1) * kCellThreads + threadIdx.x]);
        } else {
          s.list[leaf_slot] = (uint32_t)li | ((uint32_t)dl << 11) | (x << 16);
          ++leaf_slot;
        }
        put_cell(ci, kk[j], d, t0 + li, fc);
      }
    }
  }
  __syncthreads();
  if (!listed) nlist = (int)*s.nleaf;
  // the list shares its space with the records: each thread keeps its entries (at most
  // IPT: a tile starts at most one leaf a particle) and the keys they start at
  uint32_t mine[IPT];
  uint64_t my_key[IPT];
#pragma unroll
  for (int k = 0; k < IPT; ++k) {
    const int x = threadIdx.x + k * kCellThreads;
    mine[k] = x < nlist ? s.list[x] : 0u;
  }
#pragma unroll
  for (int k = 0; k < IPT; ++k) {
    const int x = threadIdx.x + k * kCellThreads, li = mine[k] & 0x7ff;
    my_key[k] = x < nlist && li < T ? keys[t0 + li] : 0ull;
  }
  __syncthreads();

  // the cursors and the list are dead: the particle records (tile and
  // halo) take their place, in batched loads
  for (int x0 = 0; x0 < span; x0 += kRecBatch * kCellThreads) {
    float4 r[kRecBatch];
#pragma unroll
    for (int u = 0; u < kRecBatch; ++u) {
      const int x = x0 + u * kCellThreads + threadIdx.x;
      r[u] = sorted[t0 + (x < span ? x : span - 1)];
    }
#pragma unroll
    for (int u = 0; u < kRecBatch; ++u) {
      const int x = x0 + u * kCellThreads + threadIdx.x;
      if (x < span) s.rec[x] = r[u];
    }
  }
  __syncthreads();

  // one lane per cell (leaf, if they are not all listed); particles read from LDS
  const double lo[3] = {box[4 * tr.b + 0], box[4 * tr.b + 1], box[4 * tr.b + 2]};
  const double side = box[4 * tr.b + 3];
#pragma unroll 1
  for (int k = 0; k < IPT; ++k) {
    const int x0 = threadIdx.x + k * kCellThreads;
    if (x0 >= nlist) break;
    // this thread's next entry; the rest move down (constant register indices)
    const uint32_t le = mine[0];
    const uint64_t key = my_key[0];
#pragma unroll
    for (int j = 0; j + 1 < IPT; ++j) {
      mine[j] = mine[j + 1];
      my_key[j] = my_key[j + 1];
    }
    const int li = le & 0x7ff;
    const int dl = (le >> 11) & 31;
    if (dl > kMaxDepth || li >= T) {  // cannot happen: entries come from the loops above
      internal = true;
      continue;
    }
    const uint32_t ci = s.lvl[dl] + (listed ? (uint32_t)x0 : le >> 16);
    if ((int64_t)ci >= c_max) {
      internal = true;
      continue;
    }
    const int64_t i = t0 + li;
    if (listed) {
      const bool leaf = (le >> 31) == 0;
      // (an internal cell's depth is below kMaxDepth)
      put_cell(ci, key, dl, i,
               leaf ? -1 : (int32_t)(s.lvl[min(dl + 1, kMaxDepth)] + ((le >> 16) & 0x7fffu)));
      if (!leaf) continue;
    }
    const int64_t e = leaf_end_fast(s, keys, n, nl, t0, T, li, dl);
    cell_count[ci] = (int32_t)(e - i);
    const int sh = kMaxDepth - dl;
    uint32_t ijk[3];
    if (hilbert) {
      cell_coords(key >> (3 * sh), dl, true, ijk);
    } else {
      ijk[0] = compact3(key >> 2) >> sh;
      ijk[1] = compact3(key >> 1) >> sh;
      ijk[2] = compact3(key) >> sh;
    }
    const int64_t e_lds = min(e, t0 + (int64_t)span);
    if constexpr (!MIXED) {
      double *com = static_cast<double *>(com_v);
      double *quad = static_cast<double *>(quad_v);
      const double h = ldexp(side, -dl);
      const double off[3] = {((double)ijk[0] + 0.5) * h, ((double)ijk[1] + 0.5) * h,
                             ((double)ijk[2] + 0.5) * h};
      LeafSums acc = {0.0, {0.0, 0.0, 0.0}, {0.0, 0.0, 0.0, 0.0, 0.0, 0.0}};
      for (int64_t q = i; q < e_lds; ++q) leaf_add(acc, s.rec[q - t0], lo, off);
      // only a saturated depth-21 leaf reaches past the staged halo
      for (int64_t q = e_lds; q < e; ++q) leaf_add(acc, sorted[q], lo, off);
      double cm[4], qd[6];
      leaf_finish(acc, cm, qd);
      double2 *cd = reinterpret_cast<double2 *>(com + 4 * (int64_t)ci);
      cd[0] = make_double2(cm[0], cm[1]);
      cd[1] = make_double2(cm[2], cm[3]);
      double2 *qq = reinterpret_cast<double2 *>(quad + 6 * (int64_t)ci);
      qq[0] = make_double2(qd[0], qd[1]);
      qq[1] = make_double2(qd[2], qd[3]);
      qq[2] = make_double2(qd[4], qd[5]);
    } else {
      float *com = static_cast<float *>(com_v);
      float *quad = static_cast<float *>(quad_v);
      const double scale = 2097152.0 / side;
      const uint32_t base[3] = {ijk[0] << sh, ijk[1] << sh, ijk[2] << sh};
      const float half = ldexpf(1.0f, sh - 1);
      LeafSumsF acc;
#pragma unroll
      for (int k = 0; k < 10; ++k) acc.s[k] = acc.c[k] = 0.0f;
      for (int64_t q = i; q < e_lds; ++q) leaf_add_f(acc, s.rec[q - t0], lo, scale, base, half, dl);
      for (int64_t q = e_lds; q < e; ++q) leaf_add_f(acc, sorted[q], lo, scale, base, half, dl);
      float cm[4], qd[6], mlo;
      leaf_finish_f(acc, cm, mlo, qd);
      // stored in absolute units: scaling by the side (a power of two) is exact
      const float l = ldexpf((float)side, -dl);
      reinterpret_cast<float4 *>(com)[ci] = make_float4(cm[0] * l, cm[1] * l, cm[2] * l, cm[3]);
      const float l2 = l * l;
      float2 *qq = reinterpret_cast<float2 *>(quad + 6 * (int64_t)ci);
      qq[0] = make_float2(qd[0] * l2, qd[1] * l2);
      qq[1] = make_float2(qd[2] * l2, qd[3] * l2);
      qq[2] = make_float2(qd[4] * l2, qd[5] * l2);
      m_lo[ci] = mlo;
    }
  }
  if (__ballot(internal) != 0 && lane_id() == 0) atomicOr(status_word, TB_STATUS_INTERNAL);
}

hipError_t launch_cell_scan(const Plan &p, const Work &w, const tb_tree &out,
                            int64_t *cell_offsets, hipStream_t s) {
  if (few_tiles(p)) return hipSuccess;
  const int gy = p.nsets < 65535 ? p.nsets : 65535;
  if (p.nsets == 1)
    k_cell_scan<1024><<<dim3(kLevels, 1), 1024, 0, s>>>(w.cell_cnt, p.cell_tiles, w.tile_start,
                                                       p.nsets, w.cell_excl, w.set_tot);
  else
    k_cell_scan<256><<<dim3(kLevels, gy), 256, 0, s>>>(w.cell_cnt, p.cell_tiles, w.tile_start,
                                                      p.nsets, w.cell_excl, w.set_tot);
  if (p.nsets <= 64) {
    k_set_scan_wave<<<1, 64, 0, s>>>(w.set_tot, p.nsets, w.set_cells, w.lvl_off, out.level_offset,
                                     cell_offsets, out.n_cells, w.par_start, w.box, out.box_out);
  } else {
    const int t = p.nsets <= kFewSets ? 64 : 256, g = (p.nsets + t - 1) / t;
    (t == 64 ? k_set_sums<64> : k_set_sums<256>)<<<g, t, 0, s>>>(w.set_tot, p.nsets, w.set_wg);
    (t == 64 ? k_set_scan_wg<64> : k_set_scan_wg<256>)<<<g, t, 0, s>>>(
        w.set_tot, p.nsets, w.set_wg, w.set_cells, w.lvl_off, out.level_offset, cell_offsets,
        out.n_cells, w.par_start, w.box, out.box_out);
  }
  return hipGetLastError();
}

// The runs and tiles left to the second launch are listed in the look-back words' space:
// at most n / (kRunCap + 1) runs, and as many tiles as there are.
static ReorderArgs reorder_args(const Plan &p, const Work &w, const tb_tree &out) {
  ReorderArgs g;
  g.order = reinterpret_cast<const int32_t *>(sorted_order(p, w, out));
  g.packed = w.packed;
  g.n = p.n;
  g.nl = p.n_leaf;
  g.skip = p.skip_bits;
  g.hilbert = (p.flags & TB_HILBERT) ? 1 : 0;
  g.tile_start = w.tile_start;
  g.tile_set = w.tile_set;
  g.set_off = w.set_off;
  g.nsets = p.nsets;
  g.box = w.box;
  g.cell_tiles = p.cell_tiles;
  g.full = w.counters + kFullSortCounter;
  g.oversize = p.set_index_bits ? w.counters + kOversizeCounter : nullptr;
  g.n_runs = w.counters + kRunCounter;
  g.n_run_tiles = w.counters + kRunTileCounter;
  g.runs = reinterpret_cast<int32_t *>(w.status0);
  g.run_tiles = reinterpret_cast<int32_t *>(w.status1);
  g.sorted = w.sorted;
  g.keys = sorted_keys(p, w);
  g.key_out = out.key_sorted;
  g.perm = out.perm;
  g.pos_sorted = out.pos_sorted;
  g.mass_sorted = out.mass_sorted;
  g.ad = w.ad;
  g.tile_cnt = w.cell_cnt;
  g.status_word = out.status;
  return g;
}

template <int IPT>
static hipError_t reorder_t(const Plan &p, const Work &w, const tb_tree &out, hipStream_t s) {
  auto k = reorder_finishes(p.n_leaf) ? k_reorder<true, IPT> : k_reorder<false, IPT>;
  k<<<(unsigned)p.cell_tiles, kCellThreads, window_lds_bytes(p.n_leaf, p.cell_tile), s>>>(
      reorder_args(p, w, out));
  return hipGetLastError();
}

hipError_t launch_reorder(const Plan &p, const Work &w, const tb_tree &out, hipStream_t s) {
  return p.cell_tile == kCellTile ? reorder_t<kCellIpt>(p, w, out, s)
                                  : reorder_t<kSmallIpt>(p, w, out, s);
}

hipError_t launch_runs(const Plan &p, const Work &w, const tb_tree &out, hipStream_t s) {
  const ReorderArgs g = reorder_args(p, w, out);
  const int64_t most = p.n / (kRunCap + 1);
  // too few particles for a run that long, or sorted by their whole keys (or no run that
  // long is left)
  if (most == 0 || !reorder_finishes(p.n_leaf) || one_tile(p)) return hipSuccess;
  // small grids, which return at once in the common case that nothing is listed (1856 runs
  // of 2^26 particles in 512 workgroups 47 us, in 256 65 us)
  const int64_t run_wgs = p.n < (int64_t{1} << 22) ? 256 : 512;
  k_sort_runs<<<(unsigned)(most < run_wgs ? most : run_wgs), kRunThreads, 0, s>>>(
      g, reinterpret_cast<int32_t *>(w.vals1), w.keys0, w.keys1);
  auto k = p.cell_tile == kCellTile ? k_reorder_again<kCellIpt> : k_reorder_again<kSmallIpt>;
  k<<<(unsigned)(p.cell_tiles < 512 ? p.cell_tiles : 512), kCellThreads,
      window_lds_bytes(p.n_leaf, p.cell_tile), s>>>(g);
  return hipGetLastError();
}

// Largest dynamic LDS a workgroup may use on the current device (cached per
// device), after opting the cell kernels in to it.
size_t cell_lds_limit() {
  static int cached_dev = -1;
  static size_t cached = 0;
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return 0;
  if (dev != cached_dev) {
    int v = 0;
    if (hipDeviceGetAttribute(&v, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess) return 0;
    const int want = (int)cell_emit_lds(TB_MAX_NLEAF, kCellTile);
    const int opt = v < want ? v : want;
    const void *kernels[] = {
        reinterpret_cast<const void *>(k_cell_emit<false, kCellIpt>),
        reinterpret_cast<const void *>(k_cell_emit<true, kCellIpt>),
        reinterpret_cast<const void *>(k_cell_emit<false, kSmallIpt>),
        reinterpret_cast<const void *>(k_cell_emit<true, kSmallIpt>),
        reinterpret_cast<const void *>(k_reorder<true, kCellIpt>),
        reinterpret_cast<const void *>(k_reorder<false, kCellIpt>),
        reinterpret_cast<const void *>(k_reorder<true, kSmallIpt>),
        reinterpret_cast<const void *>(k_reorder<false, kSmallIpt>),
        reinterpret_cast<const void *>(k_reorder_again<kCellIpt>),
        reinterpret_cast<const void *>(k_reorder_again<kSmallIpt>)};
    for (const void *k : kernels)
      (void)hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, opt);
    cached = (size_t)v;
    cached_dev = dev;
  }
  return cached;
}

hipError_t launch_cell_emit(const Plan &p, const Work &w, const tb_tree &out,
                            int64_t *cell_offsets, hipStream_t s) {
  const SetScan scan = {few_tiles(p) ? w.cell_cnt : nullptr,
                        w.cell_excl,
                        w.set_cells,
                        w.lvl_off,
                        out.level_offset,
                        cell_offsets,
                        out.n_cells,
                        w.par_start,
                        w.box,
                        out.box_out};
  const size_t lds = emit_lds_bytes(p.n_leaf, p.cell_tile);
  const bool mixed = (p.flags & 0xffu) == TB_MIXED;
  auto k = p.cell_tile == kCellTile
               ? (mixed ? k_cell_emit<true, kCellIpt> : k_cell_emit<false, kCellIpt>)
               : (mixed ? k_cell_emit<true, kSmallIpt> : k_cell_emit<false, kSmallIpt>);
  k<<<(unsigned)p.cell_tiles, kCellThreads, lds, s>>>(
      sorted_keys(p, w), w.ad, p.n_leaf, w.cell_excl, p.cell_tiles, w.tile_start, w.tile_set,
      w.set_off, p.nsets, w.lvl_off, w.box, w.sorted, out.cell_key, out.cell_level,
      out.cell_first, out.cell_count, out.child_ptr, out.com, out.quad, w.m_lo,
      owned_parents(p) ? nullptr : w.head_parent,
      p.c_max, (p.flags & TB_HILBERT) ? 1 : 0, out.status, scan);
  return hipGetLastError();
}

// The larger of the two cell kernels' LDS needs for this n_leaf and tile.
size_t cell_emit_lds(int nl, int cell_tile) {
  const size_t a = emit_lds_bytes(nl, cell_tile), b = window_lds_bytes(nl, cell_tile);
  return a > b ? a : b;
}

}  // namespace tb
