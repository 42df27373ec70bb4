// tb_parents.hip -- parents, deepest first (Sec. 2.3.2, Algorithm 2), with their counts,
// child links and moments: by the tiles of particles that hold them, or, where leaves are
// very small, one launch a depth.
//
// Algorithm 2 scans the depth-(d+1) cells in key order and hangs each one on
// the parent whose key is its own key shifted right by three bits, opening a
// new parent whenever that key changes; a parent's centre of mass (and, the
// paper notes, any higher multipole) is computed from its children once they
// are all registered.  In the (depth, key)-ordered array the children of a
// depth-d cell are one contiguous run at depth d+1, and the cell placement pass
// already recorded each internal cell's first child and, for that first child,
// the slot of its parent.  Two ways to go up the tree (owned_parents has the rule
// between them): a few launches in which every tile of particles, then every group of
// tiles, builds the cells it holds entirely (second half of this file), and, for very
// small leaves, one launch per depth: the depth-(d+1) cells (and the
// parent slots of their first children) are staged through LDS in key order; a
// child whose key, shifted right by three, differs from its predecessor's --
// the boundary test of Algorithm 2 -- opens the run of its siblings.  The
// openers of a chunk are packed to the low threads, each of which combines its
// run into the parent:
//
//   M   = sum M_c
//   com = sum M_c (com_c + s_c) / M
//   Q   = sum [Q_c + M_c (3 d_a d_b - |d|^2 delta_ab)],  d = com_c + s_c - com
//
// where s_c = +-l/4 per axis is the child centre relative to the parent centre
// (l the parent side; the octant bit picks the sign), so every quantity stays
// in a cell-relative frame.
#include "tb_internal.h"
#include "tb_moments.h"
#include "tb_tiles.h"

namespace tb {

constexpr int kChunk = kParentThreads;  // children staged per workgroup step
static_assert(kChunk == kParentThreads, "one staged child (and parent slot) per thread");
constexpr int kHalo = 7;                 // a parent has at most 8 children

// A set's parents [P0, P1) and children [P1, L2) at one depth, the first parent
// chunk of the set (row_b) and the side of its root box.
struct SetBounds {
  int64_t P0, P1, L2, row_b;
  double side;
};

__device__ inline SetBounds set_bounds(int b, int depth, const int64_t *row,
                                       const int64_t *level_offset, const double *box) {
  const int64_t *lo_b = level_offset + b * (kLevels + 1);
  return {lo_b[depth], lo_b[depth + 1], lo_b[depth + 2], row[b], box[4 * b + 3]};
}

// Packs the chunk positions of the run openers (a child at or past L1 whose
// key >> 3 differs from the previous child's) into s_open and returns their
// number.  s_key holds the keys of [base - 1, base + kChunk + kHalo); zero
// outside [L1, L2).  Both barriers are block-wide.
__device__ inline int pack_openers(const uint64_t *s_key, int64_t base, int64_t L1, int64_t L2,
                                   int *s_wop, uint16_t *s_open) {
  const int t = threadIdx.x;
  const int64_t c = base + t;
  const bool op = c < L2 && (c == L1 || (s_key[t] >> 3) != (s_key[t + 1] >> 3));
  const uint64_t bal = __ballot(op);
  if (lane_id() == 0) s_wop[t >> 6] = __popcll(bal);
  __syncthreads();
  int before = 0, total = 0;
#pragma unroll
  for (int w = 0; w < kParentThreads / 64; ++w) {
    const int v = s_wop[w];
    before += w < (t >> 6) ? v : 0;
    total += v;
  }
  if (op) s_open[before + __popcll(bal & lanemask_lt())] = (uint16_t)t;
  __syncthreads();
  return total;
}

__global__ __launch_bounds__(kParentThreads) void k_parents_fp64(
    int depth, const int64_t *__restrict__ level_offset, const uint64_t *__restrict__ cell_key,
    int32_t *__restrict__ cell_count, int32_t *__restrict__ child_ptr,
    double *__restrict__ com, double *__restrict__ quad, const int32_t *__restrict__ head_parent,
    const double *__restrict__ box, int32_t *__restrict__ status_word, int32_t nsets,
    const int64_t *__restrict__ par_start, int hilbert) {
  __shared__ uint64_t s_key[kChunk + kHalo + 1];  // keys of [base - 1, base + kChunk + kHalo)
  __shared__ int32_t s_cnt[kChunk + kHalo];
  __shared__ int32_t s_hp[kChunk];  // parent slot of each staged first child
  __shared__ int s_wop[kParentThreads / 64];
  __shared__ uint16_t s_open[kChunk];
  __shared__ __align__(16) double s_com[(kChunk + kHalo) * 4];
  __shared__ __align__(16) double s_quad[(kChunk + kHalo) * 6];

  __shared__ int s_set;
  const int64_t *row = par_start + depth * (nsets + 1);
  const int64_t n_chunks = row[nsets];
  bool internal = false;
  // the chunk's set and its bounds: loaded once for a single set (they are the
  // same for every chunk), per chunk in a batch
  SetBounds sb = {0, 0, 0, 0, 1.0};
  if (nsets == 1) sb = set_bounds(0, depth, row, level_offset, box);
  for (int64_t ch = blockIdx.x; ch < n_chunks; ch += gridDim.x) {
    if (nsets > 1) {
      if (threadIdx.x == 0) s_set = upper_index(row, nsets + 1, ch);
      __syncthreads();
      sb = set_bounds(s_set, depth, row, level_offset, box);
    }
    const int64_t P0 = sb.P0, P1 = sb.P1;
    const int64_t L1 = P1, L2 = sb.L2;
    const double q = ldexp(sb.side, -(depth + 2));  // a quarter of the parent side
    const int64_t base = L1 + (ch - sb.row_b) * (int64_t)kChunk;
    // stage the chunk: every load is issued before the first LDS store
    const int64_t lim = min((int64_t)(kChunk + kHalo), L2 - base);
    constexpr int KN = (kChunk + kHalo + 1 + kParentThreads - 1) / kParentThreads;
    constexpr int CN = (kChunk + kHalo + kParentThreads - 1) / kParentThreads;
    constexpr int MN = ((kChunk + kHalo) * 2 + kParentThreads - 1) / kParentThreads;
    constexpr int QN = ((kChunk + kHalo) * 3 + kParentThreads - 1) / kParentThreads;
    uint64_t kv[KN];
    int32_t cv[CN];
    double2 mv[MN], qv[QN];
    const int32_t hv = base + threadIdx.x < L2 ? head_parent[base + threadIdx.x] : -1;
    const double2 *com2 = reinterpret_cast<const double2 *>(com) + 2 * base;
    const double2 *quad2 = reinterpret_cast<const double2 *>(quad) + 3 * base;
#pragma unroll
    for (int r = 0; r < KN; ++r) {
      const int x = r * kParentThreads + threadIdx.x;
      const int64_t c = base - 1 + x;
      kv[r] = (x < kChunk + kHalo + 1 && c >= L1 && c < L2) ? cell_key[c] : 0ull;
    }
#pragma unroll
    for (int r = 0; r < CN; ++r) {
      const int x = r * kParentThreads + threadIdx.x;
      cv[r] = x < lim ? cell_count[base + x] : 0;
    }
#pragma unroll
    for (int r = 0; r < MN; ++r) {
      const int x = r * kParentThreads + threadIdx.x;
      mv[r] = x < 2 * lim ? com2[x] : make_double2(0.0, 0.0);
    }
#pragma unroll
    for (int r = 0; r < QN; ++r) {
      const int x = r * kParentThreads + threadIdx.x;
      qv[r] = x < 3 * lim ? quad2[x] : make_double2(0.0, 0.0);
    }
#pragma unroll
    for (int r = 0; r < KN; ++r) {
      const int x = r * kParentThreads + threadIdx.x;
      if (x < kChunk + kHalo + 1) s_key[x] = kv[r];  // 0 never matches a parent key
    }
#pragma unroll
    for (int r = 0; r < CN; ++r) {
      const int x = r * kParentThreads + threadIdx.x;
      if (x < lim) s_cnt[x] = cv[r];
    }
    s_hp[threadIdx.x] = hv;
#pragma unroll
    for (int r = 0; r < MN; ++r) {
      const int x = r * kParentThreads + threadIdx.x;
      if (x < 2 * lim) reinterpret_cast<double2 *>(s_com)[x] = mv[r];
    }
#pragma unroll
    for (int r = 0; r < QN; ++r) {
      const int x = r * kParentThreads + threadIdx.x;
      if (x < 3 * lim) reinterpret_cast<double2 *>(s_quad)[x] = qv[r];
    }
    __syncthreads();

    const int n_open = pack_openers(s_key, base, L1, L2, s_wop, s_open);
    if ((int)threadIdx.x < n_open) {
      const int t = s_open[threadIdx.x];
      const uint64_t kp = s_key[t + 1] >> 3;
      const int64_t pc = s_hp[t];
      int nch = 0;
      while (nch < 8 && t + nch < lim && (s_key[t + nch + 1] >> 3) == kp) ++nch;
      if (pc < P0 || pc >= P1) {
        internal = true;
      } else {
        double M = 0.0, S0 = 0.0, S1 = 0.0, S2 = 0.0;
        int64_t cnt = 0;
        uint32_t octs = 0;  // 3 bits per child
        for (int k = 0; k < nch; ++k) {
          const int x = t + k;
          const uint32_t o = child_octant(s_key[x + 1], depth + 1, hilbert != 0);
          octs |= o << (3 * k);
          const double mc = s_com[4 * x + 3];
          M += mc;
          S0 += mc * (s_com[4 * x + 0] + ((o & 4u) ? q : -q));
          S1 += mc * (s_com[4 * x + 1] + ((o & 2u) ? q : -q));
          S2 += mc * (s_com[4 * x + 2] + ((o & 1u) ? q : -q));
          cnt += s_cnt[x];
        }
        const double cx = S0 / M, cy = S1 / M, cz = S2 / M;
        double Q[6] = {0, 0, 0, 0, 0, 0};
        for (int k = 0; k < nch; ++k) {
          const int x = t + k;
          const uint32_t o = (octs >> (3 * k)) & 7u;
          const double mc = s_com[4 * x + 3];
          const double d0 = s_com[4 * x + 0] + ((o & 4u) ? q : -q) - cx;
          const double d1 = s_com[4 * x + 1] + ((o & 2u) ? q : -q) - cy;
          const double d2 = s_com[4 * x + 2] + ((o & 1u) ? q : -q) - cz;
          const double dd = d0 * d0 + d1 * d1 + d2 * d2;
          Q[0] += s_quad[6 * x + 0] + mc * (3.0 * d0 * d0 - dd);
          Q[1] += s_quad[6 * x + 1] + mc * (3.0 * d0 * d1);
          Q[2] += s_quad[6 * x + 2] + mc * (3.0 * d0 * d2);
          Q[3] += s_quad[6 * x + 3] + mc * (3.0 * d1 * d1 - dd);
          Q[4] += s_quad[6 * x + 4] + mc * (3.0 * d1 * d2);
          Q[5] += s_quad[6 * x + 5] + mc * (3.0 * d2 * d2 - dd);
        }
        cell_count[pc] = (int32_t)cnt;
        child_ptr[2 * pc + 1] = nch;
        double2 *cd = reinterpret_cast<double2 *>(com + 4 * pc);
        cd[0] = make_double2(cx, cy);
        cd[1] = make_double2(cz, M);
        double2 *qd = reinterpret_cast<double2 *>(quad + 6 * pc);
        qd[0] = make_double2(Q[0], Q[1]);
        qd[1] = make_double2(Q[2], Q[3]);
        qd[2] = make_double2(Q[4], Q[5]);
      }
    }
    __syncthreads();
  }
  if (__ballot(internal) != 0 && lane_id() == 0) atomicOr(status_word, TB_STATUS_INTERNAL);
}

// Mixed precision: the same combination in FP32 with Kahan-compensated sums,
// in units of the parent side (a child's frame maps to the parent's by an
// exact halving and a shift of +-1/4).  The stored moments are in absolute
// units; converting by powers of two is exact.  Each cell's mass also carries
// its compensation term (m_lo) so that the mass stays correctly rounded at
// every depth.
__device__ __forceinline__ void kahan_add_p(float &sum, float &comp, float x) {
  const float y = x - comp;
  const float t = sum + y;
  comp = (t - sum) - y;
  sum = t;
}

__global__ __launch_bounds__(kParentThreads) void k_parents_mixed(
    int depth, const int64_t *__restrict__ level_offset, const uint64_t *__restrict__ cell_key,
    int32_t *__restrict__ cell_count, int32_t *__restrict__ child_ptr,
    float *__restrict__ com, float *__restrict__ quad, float *__restrict__ m_lo,
    const int32_t *__restrict__ head_parent, const double *__restrict__ box,
    int32_t *__restrict__ status_word, int32_t nsets, const int64_t *__restrict__ par_start,
    int hilbert) {
  __shared__ uint64_t s_key[kChunk + kHalo + 1];
  __shared__ int32_t s_cnt[kChunk + kHalo];
  __shared__ int32_t s_hp[kChunk];
  __shared__ int s_wop[kParentThreads / 64];
  __shared__ uint16_t s_open[kChunk];
  __shared__ float4 s_com[kChunk + kHalo];
  __shared__ __align__(16) float s_quad[(kChunk + kHalo) * 6];
  __shared__ float s_mlo[kChunk + kHalo];

  __shared__ int s_set;
  const int64_t *row = par_start + depth * (nsets + 1);
  const int64_t n_chunks = row[nsets];
  bool internal = false;
  SetBounds sb = {0, 0, 0, 0, 1.0};
  if (nsets == 1) sb = set_bounds(0, depth, row, level_offset, box);
  for (int64_t ch = blockIdx.x; ch < n_chunks; ch += gridDim.x) {
    if (nsets > 1) {
      if (threadIdx.x == 0) s_set = upper_index(row, nsets + 1, ch);
      __syncthreads();
      sb = set_bounds(s_set, depth, row, level_offset, box);
    }
    const int64_t P0 = sb.P0, P1 = sb.P1;
    const int64_t L1 = P1, L2 = sb.L2;
    const float lc = ldexpf((float)sb.side, -(depth + 1));  // child side
    const float lp = 2.0f * lc;                             // parent side
    const float inv_lc = 1.0f / lc, inv_lc2 = inv_lc * inv_lc;
    const int64_t base = L1 + (ch - sb.row_b) * (int64_t)kChunk;
    const int64_t lim = min((int64_t)(kChunk + kHalo), L2 - base);
    constexpr int KN = (kChunk + kHalo + 1 + kParentThreads - 1) / kParentThreads;
    constexpr int CN = (kChunk + kHalo + kParentThreads - 1) / kParentThreads;
    constexpr int QN = ((kChunk + kHalo) * 3 + kParentThreads - 1) / kParentThreads;
    uint64_t kv[KN];
    int32_t cv[CN];
    const int32_t hv = base + threadIdx.x < L2 ? head_parent[base + threadIdx.x] : -1;
    float4 mv[CN];
    float lv[CN];
    float2 qv[QN];
    const float2 *quad2 = reinterpret_cast<const float2 *>(quad) + 3 * base;
#pragma unroll
    for (int r = 0; r < KN; ++r) {
      const int x = r * kParentThreads + threadIdx.x;
      const int64_t c = base - 1 + x;
      kv[r] = (x < kChunk + kHalo + 1 && c >= L1 && c < L2) ? cell_key[c] : 0ull;
    }
#pragma unroll
    for (int r = 0; r < CN; ++r) {
      const int x = r * kParentThreads + threadIdx.x;
      const int64_t c = base + (x < lim ? x : lim - 1);
      cv[r] = cell_count[c];
      mv[r] = reinterpret_cast<const float4 *>(com)[c];
      lv[r] = m_lo[c];
    }
#pragma unroll
    for (int r = 0; r < QN; ++r) {
      const int x = r * kParentThreads + threadIdx.x;
      qv[r] = quad2[x < 3 * lim ? x : 3 * lim - 1];
    }
#pragma unroll
    for (int r = 0; r < KN; ++r) {
      const int x = r * kParentThreads + threadIdx.x;
      if (x < kChunk + kHalo + 1) s_key[x] = kv[r];
    }
#pragma unroll
    for (int r = 0; r < CN; ++r) {
      const int x = r * kParentThreads + threadIdx.x;
      if (x < lim) {
        s_cnt[x] = cv[r];
        s_com[x] = mv[r];
        s_mlo[x] = lv[r];
      }
    }
    s_hp[threadIdx.x] = hv;
#pragma unroll
    for (int r = 0; r < QN; ++r) {
      const int x = r * kParentThreads + threadIdx.x;
      if (x < 3 * lim) reinterpret_cast<float2 *>(s_quad)[x] = qv[r];
    }
    __syncthreads();

    const int n_open = pack_openers(s_key, base, L1, L2, s_wop, s_open);
    if ((int)threadIdx.x < n_open) {
      const int t = s_open[threadIdx.x];
      const uint64_t kp = s_key[t + 1] >> 3;
      const int64_t pc = s_hp[t];
      int nch = 0;
      while (nch < 8 && t + nch < lim && (s_key[t + nch + 1] >> 3) == kp) ++nch;
      if (pc < P0 || pc >= P1) {
        internal = true;
      } else {
        float M = 0.f, Mc = 0.f, S[3] = {0.f, 0.f, 0.f}, Sc[3] = {0.f, 0.f, 0.f};
        int64_t cnt = 0;
        uint32_t octs = 0;  // 3 bits per child
        for (int k = 0; k < nch; ++k) {
          const int x = t + k;
          const uint32_t o = child_octant(s_key[x + 1], depth + 1, hilbert != 0);
          octs |= o << (3 * k);
          const float4 cm = s_com[x];
          const float up[3] = {0.5f * (cm.x * inv_lc) + ((o & 4u) ? 0.25f : -0.25f),
                               0.5f * (cm.y * inv_lc) + ((o & 2u) ? 0.25f : -0.25f),
                               0.5f * (cm.z * inv_lc) + ((o & 1u) ? 0.25f : -0.25f)};
          kahan_add_p(M, Mc, cm.w);
          kahan_add_p(M, Mc, s_mlo[x]);
#pragma unroll
          for (int a = 0; a < 3; ++a) kahan_add_p(S[a], Sc[a], cm.w * up[a]);
          cnt += s_cnt[x];
        }
        const float cx = S[0] / M, cy = S[1] / M, cz = S[2] / M;
        float Q[6] = {0, 0, 0, 0, 0, 0}, Qc[6] = {0, 0, 0, 0, 0, 0};
        for (int k = 0; k < nch; ++k) {
          const int x = t + k;
          const uint32_t o = (octs >> (3 * k)) & 7u;
          const float4 cm = s_com[x];
          const float mc = cm.w;
          const float d0 = 0.5f * (cm.x * inv_lc) + ((o & 4u) ? 0.25f : -0.25f) - cx;
          const float d1 = 0.5f * (cm.y * inv_lc) + ((o & 2u) ? 0.25f : -0.25f) - cy;
          const float d2 = 0.5f * (cm.z * inv_lc) + ((o & 1u) ? 0.25f : -0.25f) - cz;
          const float dd = d0 * d0 + d1 * d1 + d2 * d2;
          const float qs = 0.25f * inv_lc2;  // child units -> parent units
          kahan_add_p(Q[0], Qc[0], s_quad[6 * x + 0] * qs + mc * (3.0f * d0 * d0 - dd));
          kahan_add_p(Q[1], Qc[1], s_quad[6 * x + 1] * qs + mc * (3.0f * d0 * d1));
          kahan_add_p(Q[2], Qc[2], s_quad[6 * x + 2] * qs + mc * (3.0f * d0 * d2));
          kahan_add_p(Q[3], Qc[3], s_quad[6 * x + 3] * qs + mc * (3.0f * d1 * d1 - dd));
          kahan_add_p(Q[4], Qc[4], s_quad[6 * x + 4] * qs + mc * (3.0f * d1 * d2));
          kahan_add_p(Q[5], Qc[5], s_quad[6 * x + 5] * qs + mc * (3.0f * d2 * d2 - dd));
        }
        cell_count[pc] = (int32_t)cnt;
        child_ptr[2 * pc + 1] = nch;
        reinterpret_cast<float4 *>(com)[pc] = make_float4(cx * lp, cy * lp, cz * lp, M);
        const float lp2 = lp * lp;
        float2 *qd = reinterpret_cast<float2 *>(quad + 6 * pc);
        qd[0] = make_float2(Q[0] * lp2, Q[1] * lp2);
        qd[1] = make_float2(Q[2] * lp2, Q[3] * lp2);
        qd[2] = make_float2(Q[4] * lp2, Q[5] * lp2);
        m_lo[pc] = -Mc;
      }
    }
    __syncthreads();
  }
  if (__ballot(internal) != 0 && lane_id() == 0) atomicOr(status_word, TB_STATUS_INTERNAL);
}

// ---------------------------------------------------------------------------
// parents by ownership: a few launches for all depths
// ---------------------------------------------------------------------------
// A cell belongs to the tile that holds its first particle, and a cell whose particles
// all lie in its tile needs nothing from another one.  So one wave per tile builds
// those, deepest first (k_tile_parents); what is left are the cells that reach past
// their tile's end, at most one a depth and tile.  k_group_parents does the same with
// groups of 32 tiles for the cells that end inside their group, then with groups of 32
// groups, until one holds every tile.
//
// Eight lanes build a parent, one a child, so a step is one round of loads and not a
// loop over the children (seven on average), and a wave's step is eight parents, about
// what a tile has at a depth.  The lanes stage what they loaded in LDS, and each of the
// first six sums one component over the children in key order, which gives exactly the
// sums of a loop over them.
//
// A tile's steps follow from one another (a step is some 1.5 us), so few tiles are bound
// by that latency and many by the bytes of the cells, once in and the parents out.  us
// for all parents, by depth / so: 1000 particles 48 / 8, 65536 62 / 34, 2e6 (n_leaf 10)
// 122 / 82, 2^24 217 / 188 (118 of it the tiles), 2^26 clustered, n_leaf 8, 985 / 917;
// 300 small sets 124 / 50.
constexpr int kGroupUnits = 32;
constexpr int kGroupThreads = 8 * kGroupUnits;

struct ParentArgs {
  const uint64_t *key;
  int32_t *count, *child;
  void *com, *quad;
  float *m_lo;
  int64_t n_cells;
  int hilbert;
};

template <bool MIXED>
struct Combine;

// What the 64 lanes of a wave stage of their children.
template <>
struct Combine<false> {
  using T = double;
  struct Lds {
    double v[64][11];  // mass, com + shift, then the quadrupole's terms (one column of padding)
  };
};
template <>
struct Combine<true> {
  using T = float;
  struct Lds {
    float v[64][11];  // the same, and the mass's compensation
  };
};

__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// The eight lanes of each group of eight build parent pc (< 0: nothing to do) at depth d
// from its children, which start at cell fc.  A parent with key end_key >> (63 - 3 d)
// (end: there is a particle past what this launch's unit owns, with that key) has
// particles beyond and is left alone; returns whether this lane's is one.
template <bool MIXED>
__device__ inline bool combine_children(const ParentArgs &g, typename Combine<MIXED>::Lds &L,
                                        int64_t pc, int64_t fc, int d, double side, bool end,
                                        uint64_t end_key) {
  using T = typename Combine<MIXED>::T;
  const int lane = lane_id(), k = lane & 7, g0 = lane & ~7;
  const int64_t c = fc + k;
  const bool in = pc >= 0 && c < g.n_cells;
  const int64_t cc = in ? c : 0;
  const uint64_t key = g.key[cc];
  const int32_t cnt = g.count[cc];
  T cm[4], q[6], ml = T(0);
  if constexpr (!MIXED) {
    const double2 *com = reinterpret_cast<const double2 *>(static_cast<const double *>(g.com) + 4 * cc);
    const double2 *quad = reinterpret_cast<const double2 *>(static_cast<const double *>(g.quad) + 6 * cc);
    const double2 a = com[0], b = com[1], e = quad[0], f = quad[1], h = quad[2];
    cm[0] = a.x, cm[1] = a.y, cm[2] = b.x, cm[3] = b.y;
    q[0] = e.x, q[1] = e.y, q[2] = f.x, q[3] = f.y, q[4] = h.x, q[5] = h.y;
  } else {
    const float4 a = static_cast<const float4 *>(g.com)[cc];
    const float2 *quad = reinterpret_cast<const float2 *>(static_cast<const float *>(g.quad) + 6 * cc);
    const float2 e = quad[0], f = quad[1], h = quad[2];
    ml = g.m_lo[cc];
    cm[0] = a.x, cm[1] = a.y, cm[2] = a.z, cm[3] = a.w;
    q[0] = e.x, q[1] = e.y, q[2] = f.x, q[3] = f.y, q[4] = h.x, q[5] = h.y;
  }
  // the children: the cells from the first on whose key, shifted right by three, is the
  // first one's (the next depth's and the next set's first cells do not match)
  const uint64_t pkey = __shfl(key, g0, 64) >> 3;
  const uint64_t match = (__ballot(in && (key >> 3) == pkey) >> g0) & 0xffull;
  const int nch = __ffsll((long long)~match) - 1;
  const bool child = k < nch;
  const bool beyond = pc >= 0 && end && pkey == end_key >> (63 - 3 * d);
  const bool act = pc >= 0 && !beyond;
  const uint32_t o = child_octant(key, d + 1, g.hilbert != 0);
  T u[3];
  if constexpr (!MIXED) {
    const double sh = ldexp(side, -(d + 2));  // a quarter of the parent side
    u[0] = cm[0] + ((o & 4u) ? sh : -sh);
    u[1] = cm[1] + ((o & 2u) ? sh : -sh);
    u[2] = cm[2] + ((o & 1u) ? sh : -sh);
  } else {
    // parent units: a child's frame maps by an exact halving and a shift of a quarter
    const float lc = ldexpf((float)side, -(d + 1)), inv_lc = 1.0f / lc;
    u[0] = 0.5f * (cm[0] * inv_lc) + ((o & 4u) ? 0.25f : -0.25f);
    u[1] = 0.5f * (cm[1] * inv_lc) + ((o & 2u) ? 0.25f : -0.25f);
    u[2] = 0.5f * (cm[2] * inv_lc) + ((o & 1u) ? 0.25f : -0.25f);
  }
  T *mine = L.v[lane];
  mine[0] = cm[3];
  mine[1] = u[0];
  mine[2] = u[1];
  mine[3] = u[2];
  if (MIXED) mine[4] = ml;
  wave_lds_fence();
  // lane 0 of the eight sums the mass, lanes 1 to 3 the first moments; all terms are
  // read before the first is added
  T S = T(0), Sc = T(0);
  {
    T m[8], v[8];
#pragma unroll
    for (int x = 0; x < 8; ++x) {
      m[x] = L.v[g0 + x][0];
      v[x] = (MIXED || (k & 3) != 0) ? L.v[g0 + x][(MIXED && k == 0) ? 4 : (k & 3)] : T(1);
    }
#pragma unroll
    for (int x = 0; x < 8; ++x) {
      if constexpr (!MIXED) {
        const double t = S + m[x] * v[x];
        S = x < nch ? t : S;
      } else {
        float t = S, tc = Sc;
        if (k == 0) {
          kahan_add(t, tc, m[x]);
          kahan_add(t, tc, v[x]);
        } else {
          kahan_add_product(t, tc, m[x], v[x]);
        }
        S = x < nch ? t : S;
        Sc = x < nch ? tc : Sc;
      }
    }
  }
  // (the number of particles: every lane its child's, added up)
  int32_t n = child ? cnt : 0;
  n += __shfl_xor(n, 1, 64);
  n += __shfl_xor(n, 2, 64);
  n += __shfl_xor(n, 4, 64);
  const T M = __shfl(S, g0, 64);
  const T cj = S / M;  // lanes 1 to 3
  const T c0 = __shfl(cj, g0 + 1, 64), c1 = __shfl(cj, g0 + 2, 64), c2 = __shfl(cj, g0 + 3, 64);
  const T mc = cm[3];
  const T d0 = u[0] - c0, d1 = u[1] - c1, d2 = u[2] - c2;
  const T dd = d0 * d0 + d1 * d1 + d2 * d2;
  T qs = T(1);
  if (MIXED) {
    const float lc = ldexpf((float)side, -(d + 1)), inv_lc = 1.0f / lc;
    qs = 0.25f * (inv_lc * inv_lc);  // child units -> parent units
  }
  const T three = T(3);
  wave_lds_fence();  // the sums have read the masses
  if constexpr (!MIXED) {
    mine[0] = q[0] + mc * (three * d0 * d0 - dd);
    mine[1] = q[1] + mc * (three * d0 * d1);
    mine[2] = q[2] + mc * (three * d0 * d2);
    mine[3] = q[3] + mc * (three * d1 * d1 - dd);
    mine[4] = q[4] + mc * (three * d1 * d2);
    mine[5] = q[5] + mc * (three * d2 * d2 - dd);
  } else {
    // (fused products spelled out: the same roundings as in k_parents_mixed)
    const float s2 = fmaf(d2, d2, fmaf(d0, d0, d1 * d1));
    mine[0] = fmaf(q[0], qs, mc * fmaf(three * d0, d0, -s2));
    mine[1] = fmaf(q[1], qs, mc * (three * d0 * d1));
    mine[2] = fmaf(q[2], qs, mc * (three * d0 * d2));
    mine[3] = fmaf(q[3], qs, mc * fmaf(three * d1, d1, -s2));
    mine[4] = fmaf(mc, three * d1 * d2, q[4] * qs);
    mine[5] = fmaf(q[5], qs, mc * fmaf(three * d2, d2, -s2));
  }
  wave_lds_fence();
  T Q = T(0), Qc = T(0);
  {
    T v[8];
#pragma unroll
    for (int x = 0; x < 8; ++x) v[x] = L.v[g0 + x][k < 6 ? k : 5];
#pragma unroll
    for (int x = 0; x < 8; ++x) {
      if constexpr (!MIXED) {
        Q = x < nch ? Q + v[x] : Q;
      } else {
        float t = Q, tc = Qc;
        kahan_add(t, tc, v[x]);
        Q = x < nch ? t : Q;
        Qc = x < nch ? tc : Qc;
      }
    }
  }
  wave_lds_fence();  // the staged terms are consumed
  if (act) {
    T lp = T(1);
    if (MIXED) lp = 2.0f * ldexpf((float)side, -(d + 1));  // parent side: absolute units
    T *com = static_cast<T *>(g.com) + 4 * pc;
    if (k == 0) com[3] = M;
    if (k >= 1 && k < 4) com[k - 1] = MIXED ? cj * lp : cj;
    if (k < 6) static_cast<T *>(g.quad)[6 * pc + k] = MIXED ? Q * (lp * lp) : Q;
    if (k == 6) g.count[pc] = n;
    if (k == 7) g.child[2 * pc + 1] = nch;
    if (MIXED && k == 0) g.m_lo[pc] = (float)-Sc;
  }
  return beyond;
}

// Key of the particle past the end of a tile, if its set goes on there.
struct UnitEnd {
  bool end;
  uint64_t key;
};
__device__ inline UnitEnd unit_end(const TileRange &tr, const uint64_t *__restrict__ keys) {
  UnitEnd e;
  e.end = tr.t1 < tr.E;
  e.key = keys[e.end ? tr.t1 : tr.t0];
  return e;
}

template <bool MIXED>
__global__ __launch_bounds__(kParentThreads) void k_tile_parents(
    ParentArgs g, const uint64_t *__restrict__ keys, const uint32_t *__restrict__ excl,
    int64_t cell_tiles, const int64_t *__restrict__ tile_start,
    const int32_t *__restrict__ tile_set, const int64_t *__restrict__ set_off, int32_t nsets,
    int cell_tile, const int64_t *__restrict__ lvl_off, const double *__restrict__ box,
    const int64_t *__restrict__ n_cells, int32_t *__restrict__ left) {
  constexpr int W = kParentThreads / 64;
  __shared__ typename Combine<MIXED>::Lds s_lds[W];
  typename Combine<MIXED>::Lds &L = s_lds[threadIdx.x / 64];
  const int lane = lane_id();
  const int64_t tile = (int64_t)xcd_tile(blockIdx.x, gridDim.x) * W + threadIdx.x / 64;
  if (tile >= tile_start[nsets]) return;  // the whole wave; no barrier follows
  g.n_cells = *n_cells;
  const TileRange tr = tile_range(tile, tile_start, tile_set, set_off, cell_tile);
  const double side = box[4 * tr.b + 3];
  const UnitEnd ue = unit_end(tr, keys);
  // lane d: the cells [r0, r0 + rn) of depth d that start in the tile
  int32_t r0 = 0, rn = 0, mine = -1;
  if (lane < kLevels) {
    const int64_t *lo = lvl_off + tr.b * (kLevels + 1) + lane;
    const uint32_t *ex = excl + lane * cell_tiles + tile;
    const int64_t a = lo[0] + ex[0];
    const int64_t b = tile + 1 < tile_start[tr.b + 1] ? lo[0] + ex[1] : lo[1];
    r0 = (int32_t)a;
    rn = (int32_t)(b - a);
  }
  // depths that have cells with children (their children start in the tile as well)
  uint32_t depths = (uint32_t)__ballot(rn != 0);
  depths &= depths >> 1;
  auto first_child = [&](int d, int32_t x0) {
    const int32_t a = __shfl(r0, d, 64), n = __shfl(rn, d, 64), x = x0 + lane;
    return x < n ? g.child[2 * ((int64_t)a + x)] : -1;
  };
  int d = 31 - __clz((int)depths);  // deepest first
  int32_t ahead = depths != 0 ? first_child(d, 0) : -1;
  while (depths != 0) {
    const int32_t a = __shfl(r0, d, 64), n = __shfl(rn, d, 64);
    depths &= ~(1u << d);
    const int next = depths != 0 ? 31 - __clz((int)depths) : 0;
    int32_t fc = ahead;
    if (depths != 0) ahead = first_child(next, 0);
    for (int32_t x0 = 0; x0 < n; x0 += 64) {
      if (x0 != 0) fc = first_child(d, x0);
      uint64_t todo = __ballot(fc >= 0);
      while (todo != 0) {
        // the next eight internal cells, eight lanes each
        int src = -1;
        uint64_t rest = todo;
#pragma unroll
        for (int p = 0; p < 8; ++p) {
          if (rest != 0) {
            if (p == lane / 8) src = __ffsll((long long)rest) - 1;
            rest &= rest - 1;
          }
        }
        todo = rest;
        const int32_t pf = __shfl(fc, src < 0 ? 0 : src, 64);
        const int64_t pc = src < 0 ? -1 : (int64_t)a + x0 + src;
        const uint64_t past = __ballot(
            combine_children<MIXED>(g, L, pc, src < 0 ? 0 : pf, d, side, ue.end, ue.key));
        if (past != 0) {
          const int32_t slot = (int32_t)__shfl(pc, __ffsll((long long)past) - 1, 64);
          if (lane == d) mine = slot;
        }
      }
    }
    // the next depth's loads see these stores: a wave's accesses stay in order
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    d = next;
  }
  if (lane < kMaxDepth) left[lane * cell_tiles + tile] = mine;
}

// The cells that reach past their unit (`unit` tiles), for kGroupUnits units: those that
// end inside the group are built, the others go to left2.
template <bool MIXED>
__global__ __launch_bounds__(kGroupThreads) void k_group_parents(
    ParentArgs g, const uint64_t *__restrict__ keys, int64_t unit,
    const int64_t *__restrict__ tile_start, const int32_t *__restrict__ tile_set,
    const int64_t *__restrict__ set_off, int32_t nsets, int cell_tile,
    const double *__restrict__ box, const int64_t *__restrict__ n_cells,
    const int32_t *__restrict__ left, int64_t units,
    int32_t *__restrict__ left2, int64_t groups) {
  __shared__ typename Combine<MIXED>::Lds s_lds[kGroupThreads / 64];
  __shared__ int32_t s_pc[kMaxDepth][kGroupUnits], s_fc[kMaxDepth][kGroupUnits];
  __shared__ int32_t s_left[kMaxDepth];
  __shared__ uint32_t s_any;
  typename Combine<MIXED>::Lds &L = s_lds[threadIdx.x / 64];
  const int64_t tiles = tile_start[nsets], u0 = blockIdx.x * (int64_t)kGroupUnits;
  g.n_cells = *n_cells;
  if (threadIdx.x == 0) s_any = 0;
  if (threadIdx.x < kMaxDepth) s_left[threadIdx.x] = -1;
  __syncthreads();
  for (int x = threadIdx.x; x < kMaxDepth * kGroupUnits; x += kGroupThreads) {
    const int d = x / kGroupUnits, q = x % kGroupUnits;
    const int32_t pc = (u0 + q) * unit < tiles ? left[d * units + u0 + q] : -1;
    s_pc[d][q] = pc;
    s_fc[d][q] = pc >= 0 ? g.child[2 * (int64_t)pc] : 0;
    if (pc >= 0) atomicOr(&s_any, 1u << d);
  }
  __syncthreads();
  const uint32_t any = s_any;
  if (any != 0) {
    const int q = threadIdx.x / 8;  // this lane's unit of the group
    // the unit's and the group's last tile; a cell left over is of the set of the first
    const int64_t last = min((u0 + kGroupUnits) * unit, tiles) - 1;
    const int64_t tile = min((u0 + q + 1) * unit - 1, last);
    const int b = tile_set[tile], bl = tile_set[last];
    const double side = box[4 * b + 3];
    const UnitEnd ue = unit_end(tile_range(last, tile_start, tile_set, set_off, cell_tile), keys);
    for (int d = kMaxDepth - 1; d >= 0; --d) {
      if (!((any >> d) & 1u)) continue;
      const int64_t pc = s_pc[d][q];
      if (combine_children<MIXED>(g, L, pc, s_fc[d][q], d, side, ue.end && b == bl, ue.key))
        s_left[d] = (int32_t)pc;
      __syncthreads();  // the next depth's loads see these stores
    }
  }
  if (threadIdx.x < kMaxDepth) left2[threadIdx.x * groups + blockIdx.x] = s_left[threadIdx.x];
}

// Launches of k_group_parents, each with units of kGroupUnits times the tiles.  Tiles are
// numbered through all sets, so a set of a batch may lie over the end of any unit, however
// few particles it has: a batch goes on until one unit holds every tile (none if every
// set is one tile: n at most a tile's).  A single set's units start where it does, so it
// stops at the unit that reaches its n particles, without the tile the plan has to spare.
int group_levels(const Plan &p) {
  int levels = 0;
  int64_t units = p.cell_tiles, unit = 1;
  while (p.nsets > 1 ? p.n > p.cell_tile && units > 1 : unit * p.cell_tile < p.n) {
    units = (units + kGroupUnits - 1) / kGroupUnits;
    unit *= kGroupUnits;
    ++levels;
  }
  return levels;
}

template <bool MIXED>
static hipError_t owned_parents_t(const Plan &p, const Work &w, const tb_tree &out,
                                  hipStream_t s) {
  const ParentArgs g = {out.cell_key, out.cell_count, out.child_ptr, out.com, out.quad,
                        w.m_lo,       0,              (p.flags & TB_HILBERT) ? 1 : 0};
  const uint64_t *keys = sorted_keys(p, w);
  // the cells left over lie in the space of the tiles' cell counts and then, of the
  // groups, by turns in that of the two buffers of look-back words (84 bytes a group)
  const int32_t *left = reinterpret_cast<int32_t *>(w.cell_cnt);
  int32_t *space[2] = {reinterpret_cast<int32_t *>(w.status0),
                       reinterpret_cast<int32_t *>(w.status1)};
  constexpr int W = kParentThreads / 64;
  k_tile_parents<MIXED><<<(unsigned)((p.cell_tiles + W - 1) / W), kParentThreads, 0, s>>>(
      g, keys, w.cell_excl, p.cell_tiles, w.tile_start, w.tile_set, w.set_off, p.nsets, p.cell_tile,
      w.lvl_off, w.box, out.n_cells, reinterpret_cast<int32_t *>(w.cell_cnt));
  int64_t units = p.cell_tiles, unit = 1;
  for (int level = 0, levels = group_levels(p); level < levels; ++level) {
    const int64_t groups = (units + kGroupUnits - 1) / kGroupUnits;
    k_group_parents<MIXED><<<(unsigned)groups, kGroupThreads, 0, s>>>(
        g, keys, unit, w.tile_start, w.tile_set, w.set_off, p.nsets, p.cell_tile, w.box,
        out.n_cells, left, units, space[level % 2], groups);
    left = space[level % 2];
    units = groups;
    unit *= kGroupUnits;
  }
  return hipGetLastError();
}

// Whether the parents are built tile by tile or one launch a depth.  A wave goes through
// its tile's cells one after the other, so where leaves are so small that a tile has
// thousands, that takes longer than 21 launches; tiles of 512 have fewer.  us a build, by
// depth / by tile, Plummer (clustered): tiles of 512, n_leaf 1, 4096 particles 123 / 123
// (127 / 142), 65536 174 / 178 (177 / 197); n_leaf 4 116 / 84 (117 / 93), 159 / 135
// (164 / 141).  Tiles of 2048, n_leaf 1, 2^21 615 / 728, 2^24 3687 / 3704; n_leaf 4
// 413 / 418, 1922 / 1944; n_leaf 6 390 / 376, 1719 / 1719; n_leaf 16 358 / 339,
// 1470 / 1458.
bool owned_parents(const Plan &p) {
  return p.n_leaf >= (p.cell_tile == kSmallTile ? 4 : 6);
}

hipError_t launch_owned_parents(const Plan &p, const Work &w, const tb_tree &out, hipStream_t s) {
  return (p.flags & 0xffu) == TB_MIXED ? owned_parents_t<true>(p, w, out, s)
                                       : owned_parents_t<false>(p, w, out, s);
}

hipError_t launch_parents(const Plan &p, const Work &w, int depth, const tb_tree &out,
                          hipStream_t s) {
  // at most 8^(depth+1) children per set one depth down, in chunks of kChunk
  int64_t bound = p.c_max;
  if (depth + 1 < 10) {
    const int64_t b8 = (int64_t(1) << (3 * (depth + 1))) * p.nsets;
    if (b8 < bound) bound = b8;
  }
  int64_t blocks = (bound + kChunk - 1) / kChunk + p.nsets;
  if (blocks > 1024) blocks = 1024;
  if (blocks < 1) blocks = 1;
  if ((p.flags & 0xffu) == TB_MIXED)
    k_parents_mixed<<<(unsigned)blocks, kParentThreads, 0, s>>>(
        depth, w.lvl_off, out.cell_key, out.cell_count, out.child_ptr,
        static_cast<float *>(out.com), static_cast<float *>(out.quad), w.m_lo, w.head_parent,
        w.box, out.status, p.nsets, w.par_start, (p.flags & TB_HILBERT) ? 1 : 0);
  else
    k_parents_fp64<<<(unsigned)blocks, kParentThreads, 0, s>>>(
        depth, w.lvl_off, out.cell_key, out.cell_count, out.child_ptr,
        static_cast<double *>(out.com), static_cast<double *>(out.quad), w.head_parent, w.box,
        out.status, p.nsets, w.par_start, (p.flags & TB_HILBERT) ? 1 : 0);
  return hipGetLastError();
}

}  // namespace tb
