// tb_gravity.hip -- the gravity calculation that consumes the tree (Sec. 2.1).
//
// Barnes-Hut with Barnes' shared interaction lists: the particles of a group
// (the first cell on each path down from the root that holds at most n_crit
// particles, or is a leaf) share one list, built by one workgroup walking the
// tree from the root.  A cell C is accepted for group G when it is neither G
// nor one of its ancestors and l_C < theta * d, d the distance from C's centre
// of mass to the closest point of G's cube (eq. 1, l/d < theta, then holds for
// every particle of G).  A cell that is not accepted is opened: a leaf gives
// its particles (direct, softened terms), an internal cell its children.
//
// k_find_groups  : every internal cell holding more than n_crit particles
//                  lists those of its children that are groups (the root
//                  itself when it is one), a large group as several items.
// k_walk         : one workgroup per item at a time, the items taken from a
//                  counter.  The cells still to visit sit on an LDS stack; a
//                  round pops up to one cell per thread, tests it, and appends
//                  accepted cells, opened leaves and the children of opened
//                  cells at positions given by block-wide counts (so lists and
//                  sums come out in the same order on every run).  Once a list
//                  is nearly full, or nothing is left to visit, the listed
//                  cells and leaf particles are staged in LDS batch by batch
//                  and added to the group's particles.  FP64 throughout.
//
// The threads of an item.  A group holds anything from one particle to n_crit
// (128 on average at n_crit 512, 20 at 64), so giving every thread particles of
// its own leaves most lanes idle.  Instead the particles are spread over
// Q = ceil(P / U) lanes with U of them each, and S = T / Q such sets of lanes
// take every S-th source of a batch; U (1 to 4) is the one that wastes the
// fewest lanes.  The S partial sums of a particle are added in order at the end.
// A source is read from LDS once for U particles.
#include <cmath>

#include "tb_internal.h"
#include "tb_moments.h"

namespace tb {

constexpr int kWalkThreads = 256;
// Three waves a SIMD (168 VGPRs): held to four, the walk spills 44 registers and is
// no faster at 2^21 particles (8.0 ms either way) and slower on few groups (2^14:
// 0.30 against 0.25 ms).  Two waves measure as three: the arithmetic is bound by the
// FP64 units (5.3 cycles an instruction and SIMD where they are kept busy), not by
// latency.  128 and 512 threads: 7.8 and 10.4 ms at 2^21, 1.04 and 1.28 ms at 3e5.
constexpr int kWalkWaves = 3;
constexpr int kWalkPpt = 4;       // most group particles per thread and pass
// Cells a depth-first descent can add to the stack: 7 a level, one popped at a time.
constexpr int kStackReserve = 7 * kMaxDepth;

// LDS lists and batches of a workgroup of T threads.
template <int T>
struct WalkShape {
  static constexpr int kWaves = T / 64;
  static constexpr int kStack = T > 512 ? 8 * T : 4096;  // cells waiting to be visited
  static constexpr int kCells = 4 * T;           // accepted cells listed before they are added
  static constexpr int kLeaves = 2 * T;          // opened leaves listed
  static constexpr int kCellBatch = T / 2;       // cells staged at once, two threads each
  static constexpr int kPartBatch = T / 2 * 10 / 4;  // source particles staged at once
};

// What a lane pays for each source besides its U interactions (LDS reads, loop), in
// 1/1024ths of one interaction's time for one particle a lane: 8.06, 7.99 and 8.22 ms
// at 2^21 with 128, 400 and 0.
constexpr int kReadCost = 400;

struct GravArgs {
  const uint64_t *key;
  const int32_t *first, *count, *child;
  const double *com, *quad;
  const double *box;
  const float *pos;   // sorted positions [n][3]
  const float *mass;  // sorted masses [n]
  double theta2, eps2;  // (eps2: minus infinity stands for infinity)
  int hilbert;  // the cell keys are Peano-Hilbert keys
};

// Depth of the cell with this key (its leading 1 sits at bit 3 depth).
__device__ __forceinline__ int cell_depth(uint64_t key) {
  return (63 - __clzll((long long)key)) / 3;
}

// Geometric centre (absolute) and side of the depth-d cell with this key.
__device__ __forceinline__ void cell_centre(const GravArgs &g, uint64_t key, int d, double (&cen)[3],
                                            double &l) {
  uint32_t ijk[3];
  cell_coords(key, d, g.hilbert != 0, ijk);
  l = ldexp(g.box[3], -d);
#pragma unroll
  for (int a = 0; a < 3; ++a) cen[a] = g.box[a] + ((double)ijk[a] + 0.5) * l;
}

// counts[0]: number of groups, counts[1]: groups taken by the walk
__global__ void k_grav_init(uint32_t *__restrict__ counts, unsigned long long *__restrict__ stats) {
  if (threadIdx.x < 2) counts[threadIdx.x] = 0;
  if (stats && threadIdx.x < 2) stats[threadIdx.x] = 0;
}

// A group of more than `part` particles is several items of work (one, if the groups stay
// whole): its first slot holds the cell, the k-th after it -k.
__device__ __forceinline__ void list_group(int32_t *__restrict__ items,
                                           uint32_t *__restrict__ n_items, int32_t cell,
                                           int32_t count, int32_t part, int whole) {
  const uint32_t k = whole ? 1u : (uint32_t)((count + (int64_t)part - 1) / part);
  const uint32_t at = atomicAdd(n_items, k);
  items[at] = cell;
  for (uint32_t q = 1; q < k; ++q) items[at + q] = -(int32_t)q;
}

__global__ __launch_bounds__(256) void k_find_groups(
    const int64_t *__restrict__ n_cells, const int32_t *__restrict__ count,
    const int32_t *__restrict__ child, int32_t n_crit, int32_t part, int whole,
    int32_t *__restrict__ items, uint32_t *__restrict__ n_items) {
  const int64_t C = *n_cells;
  for (int64_t c = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; c < C;
       c += (int64_t)gridDim.x * blockDim.x) {
    const bool leaf = child[2 * c] < 0;
    if (c == 0 && (leaf || count[0] <= n_crit)) list_group(items, n_items, 0, count[0], part, whole);
    if (leaf || count[c] <= n_crit) continue;
    const int32_t f = child[2 * c], nch = child[2 * c + 1];
    for (int k = 0; k < nch; ++k) {
      const int32_t ch = f + k;
      if (child[2 * ch] < 0 || count[ch] <= n_crit)
        list_group(items, n_items, ch, count[ch], part, whole);
    }
  }
}

// 1 / sqrt(x) for x >= 0.  The hardware's approximation y has a relative error of
// at most 2^-24.  With e = 1 - x y^2 the root is y (1 - e)^(-1/2), and Newton's binomial
// series of that up to its second power, y + y e (1/2 + 3/8 e) (Householder's step of third
// order for 1 / y^2 - x), leaves little more than one rounding (measured over 2^-50 .. 2^10: 1.4e-16 at
// most and 5.3e-17 rms, where 1 / sqrt(x) has 1.7e-16 and 6.7e-17) in six
// instructions instead of some thirty.  Zero and infinity, where e is not a number,
// keep y, which is exact there; EDGE = false leaves that out for an x that is neither.
template <bool EDGE>
__device__ __forceinline__ double rsqrt_fp64(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  const double e = fma(-(x * y), y, 1.0);
  const double z = fma(y * e, fma(0.375, e, 0.5), y);
  constexpr int kZeroOrInf = (1 << 5) | (1 << 6) | (1 << 9);  // v_cmp_class bits
  return EDGE && __builtin_amdgcn_class(x, kZeroOrInf) ? y : z;
}

// A value that is the same in every lane, moved to scalar registers.
__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ uint64_t uniform(uint64_t v) {
  return ((uint64_t)(uint32_t)uniform((int)(v >> 32)) << 32) | (uint32_t)uniform((int)(uint32_t)v);
}
__device__ __forceinline__ double uniform(double v) {
  return __longlong_as_double((long long)uniform((uint64_t)__double_as_longlong(v)));
}

// Sum over the lanes below this one of v, 0 <= v < 16, and over the whole wave.
__device__ __forceinline__ int wave_excl_nibble(int v, int *total) {
  const uint64_t lt = lanemask_lt();
  int pre = 0, tot = 0;
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    const uint64_t m = __ballot((v >> b) & 1);
    pre += __popcll(m & lt) << b;
    tot += __popcll(m) << b;
  }
  *total = tot;
  return pre;
}

template <int T>
struct WalkLds {
  using W = WalkShape<T>;
  int32_t stack[W::kStack];
  int32_t cells[W::kCells];        // accepted cells
  int32_t leaves[W::kLeaves];      // opened leaves; their first particles while they are added
  int32_t lstart[W::kLeaves + 1];  // where each leaf's particles start among all listed ones
  union {
    double cell[W::kCellBatch][10];  // com (absolute) x y z, M, Q[6]
    double part[W::kPartBatch][4];   // x y z m of source particles
    double sum[T][4];                // partial sums of one of a thread's particles
  };
  int32_t pidx[W::kPartBatch];
  uint32_t w0[W::kWaves], w1[W::kWaves];
  uint32_t next;
};

// A batch's terms are summed on their own and then added, so that the sum over a
// list of thousands loses less: against 80-bit arithmetic on 6000 Plummer particles
// accelerations are off by 5.5e-16 and potentials by 1.9e-16 (2-norm), 1.15e-15 and
// 1.2e-15 when every term went to the running sum through a square root and a
// division.
template <int U>
__device__ __forceinline__ void add_sums(double (&ai)[U][4], const double (&bi)[U][4]) {
#pragma unroll
  for (int u = 0; u < U; ++u)
#pragma unroll
    for (int a = 0; a < 4; ++a) ai[u][a] += bi[u][a];
}

// Adds the accepted cells [0, n) of the list to the group's particles.
template <int T, int U, bool QUAD, bool WHOLE>
__device__ __forceinline__ void add_cells(const GravArgs &g, WalkLds<T> &L, int n,
                                          const float (&xf)[U][3], double (&ai)[U][4], int slice,
                                          int S, bool idle) {
  using W = WalkShape<T>;
  for (int c0 = 0; c0 < n; c0 += W::kCellBatch) {
    const int nc = min(W::kCellBatch, n - c0);
    __syncthreads();  // the list is complete, the previous batch consumed
    const int slot = threadIdx.x % W::kCellBatch;
    if (slot < nc) {
      const int64_t cc = L.cells[c0 + slot];
      if (threadIdx.x < W::kCellBatch) {
        const uint64_t key = g.key[cc];
        const double2 *cm = reinterpret_cast<const double2 *>(g.com + 4 * cc);
        const double2 m0 = cm[0], m1 = cm[1];
        double cen[3], l;
        cell_centre(g, key, cell_depth(key), cen, l);
        L.cell[slot][0] = cen[0] + m0.x;
        L.cell[slot][1] = cen[1] + m0.y;
        L.cell[slot][2] = cen[2] + m1.x;
        L.cell[slot][3] = m1.y;
      } else if (QUAD) {
        const double2 *qd = reinterpret_cast<const double2 *>(g.quad + 6 * cc);
        double2 *o = reinterpret_cast<double2 *>(&L.cell[slot][4]);
        const double2 q0 = qd[0], q1 = qd[1], q2 = qd[2];
        o[0] = q0;
        o[1] = q1;
        o[2] = q2;
      }
    }
    __syncthreads();
    if (idle) continue;
    double xi[U][3];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int a = 0; a < 3; ++a) xi[u][a] = (double)xf[u][a];
    double bi[U][4] = {};
    for (int k = slice; k < nc; k += S) {
      const double2 *row = reinterpret_cast<const double2 *>(L.cell[k]);
      const double2 p0 = row[0], p1 = row[1];
      const double M = p1.y;
      double2 q01, q23, q45;
      if (QUAD) {
        q01 = row[2];
        q23 = row[3];
        q45 = row[4];
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const double r0 = xi[u][0] - p0.x, r1 = xi[u][1] - p0.y, r2 = xi[u][2] - p1.x;
        const double u1 = rsqrt_fp64<true>(fma(r2, r2, fma(r1, r1, r0 * r0)));
        const double u2 = u1 * u1, u3 = u1 * u2;
        double A = M * u3;  // a -= A r
        bi[u][3] = fma(-M, u1, bi[u][3]);
        if (QUAD) {
          const double v0 = fma(q23.x, r2, fma(q01.y, r1, q01.x * r0));
          const double v1 = fma(q45.x, r2, fma(q23.y, r1, q01.y * r0));
          const double v2 = fma(q45.y, r2, fma(q45.x, r1, q23.x * r0));
          const double rqr = fma(r2, v2, fma(r1, v1, r0 * v0));
          const double B = u3 * u2, c = rqr * B;
          A = fma(2.5 * u2, c, A);
          bi[u][0] = fma(B, v0, bi[u][0]);
          bi[u][1] = fma(B, v1, bi[u][1]);
          bi[u][2] = fma(B, v2, bi[u][2]);
          bi[u][3] = fma(-0.5, c, bi[u][3]);
        }
        bi[u][0] = fma(-A, r0, bi[u][0]);
        bi[u][1] = fma(-A, r1, bi[u][1]);
        bi[u][2] = fma(-A, r2, bi[u][2]);
      }
    }
    add_sums<U>(ai, bi);
  }
}

// Particle terms of one staged batch.  SELF: the batch holds particles of the
// group, so a particle may meet itself, which gives no term (or eps^2 is zero, and
// coincident particles are at distance zero, or infinite, as every distance is then).
template <int T, int U, bool SELF>
__device__ __forceinline__ void add_batch(const WalkLds<T> &L, double eps2, int nb,
                                          const float (&xf)[U][3], const int32_t (&si)[U],
                                          double (&ai)[U][4], int slice, int S) {
  double xi[U][3];
#pragma unroll
  for (int u = 0; u < U; ++u)
#pragma unroll
    for (int a = 0; a < 3; ++a) xi[u][a] = (double)xf[u][a];
  double bi[U][4] = {};
  for (int k = slice; k < nb; k += S) {
    const double2 *row = reinterpret_cast<const double2 *>(L.part[k]);
    const double2 p0 = row[0], p1 = row[1];
    int32_t id = 0;
    if (SELF) id = L.pidx[k];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const double r0 = xi[u][0] - p0.x, r1 = xi[u][1] - p0.y, r2 = xi[u][2] - p1.x;
      double u1 = rsqrt_fp64<SELF>(fma(r2, r2, fma(r1, r1, fma(r0, r0, eps2))));
      if (SELF) u1 = id == si[u] ? 0.0 : u1;
      const double w = p1.y * u1, A = w * (u1 * u1);
      bi[u][0] = fma(-A, r0, bi[u][0]);
      bi[u][1] = fma(-A, r1, bi[u][1]);
      bi[u][2] = fma(-A, r2, bi[u][2]);
      bi[u][3] -= w;
    }
  }
  add_sums<U>(ai, bi);
}

// Adds the particles of the opened leaves [0, n) of the list; returns how many
// there are.
template <int T, int U, bool WHOLE>
__device__ __forceinline__ int add_leaves(const GravArgs &g, WalkLds<T> &L, int n, int32_t gf,
                                          int64_t gn, const float (&xf)[U][3],
                                          const int32_t (&si)[U], double (&ai)[U][4], int slice,
                                          int S, bool idle) {
  using W = WalkShape<T>;
  constexpr int R = W::kLeaves / T;
  if (n == 0) return 0;
  __syncthreads();  // the list is complete, the staged cells consumed
  // first particle and running count of every leaf, R consecutive leaves a thread
  int32_t cnt[R], mine = 0;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int x = threadIdx.x * R + r;
    const int32_t c = x < n ? L.leaves[x] : -1;
    cnt[r] = c >= 0 ? g.count[c] : 0;
    if (c >= 0) L.leaves[x] = g.first[c];
    mine += cnt[r];
  }
  const uint32_t inc = wave_inclusive_scan((uint32_t)mine);
  if (lane_id() == 63) L.w0[threadIdx.x / 64] = inc;
  __syncthreads();
  int total = 0, run = (int)inc - mine;
#pragma unroll
  for (int q = 0; q < W::kWaves; ++q) {
    const int t = (int)L.w0[q];
    run += q < (int)threadIdx.x / 64 ? t : 0;
    total += t;
  }
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int x = threadIdx.x * R + r;
    if (x <= n) L.lstart[x] = run;
    run += cnt[r];
  }
  total = uniform(total);
  if (threadIdx.x == 0) L.lstart[n] = total;
  for (int q0 = 0; q0 < total; q0 += W::kPartBatch) {
    const int nb = min(W::kPartBatch, total - q0);
    __syncthreads();  // the starts are written, the previous batch consumed
    bool own = false;
    for (int x = threadIdx.x; x < nb; x += T) {
      const int q = q0 + x;
      int lo = 0, hi = n - 1;  // the leaf holding slot q
      while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (L.lstart[mid] <= q)
          lo = mid;
        else
          hi = mid - 1;
      }
      const int64_t s = (int64_t)L.leaves[lo] + (q - L.lstart[lo]);
      const float px = g.pos[3 * s + 0], py = g.pos[3 * s + 1], pz = g.pos[3 * s + 2];
      const float pm = g.mass[s];
      double2 *o = reinterpret_cast<double2 *>(L.part[x]);
      o[0] = make_double2((double)px, (double)py);
      o[1] = make_double2((double)pz, (double)pm);
      L.pidx[x] = (int32_t)s;
      own |= s >= gf && s - gf < gn;
    }
    const bool self = __syncthreads_or(own ? 1 : 0) != 0 || !(g.eps2 > 0.0);
    if (idle) continue;
    if (self)
      add_batch<T, U, true>(L, fabs(g.eps2), nb, xf, si, ai, slice, S);
    else
      add_batch<T, U, false>(L, g.eps2, nb, xf, si, ai, slice, S);
  }
  return total;
}

// Walks the tree for the P particles from sorted position f0 on, which belong to
// group `grp` (particles [gf, gf + gn)), and writes their accelerations.
// cells, pairs: the cells and particles on the lists.
template <int T, int U, bool QUAD, bool WHOLE>
__device__ __forceinline__ void walk_pass(const GravArgs &g, WalkLds<T> &L, uint64_t gkey, int gd,
                                          const double (&gc)[3], double gh, int32_t gf, int64_t gn,
                                          int64_t f0, int P, double *__restrict__ acc,
                                          int64_t *cells, int64_t *pairs) {
  using W = WalkShape<T>;
  const int Q = (P + U - 1) / U;  // lanes of one set
  const int S = T / Q;            // sets of lanes
  const int slice = threadIdx.x / Q, lane0 = threadIdx.x - slice * Q;
  const bool idle = slice >= S;
  float xf[U][3];  // widened where they are used: half the registers during the walk
  double ai[U][4];
  int32_t si[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int k = lane0 + u * Q;
    const int64_t s = f0 + (k < P ? k : 0);
    si[u] = (int32_t)s;
#pragma unroll
    for (int a = 0; a < 3; ++a) xf[u][a] = g.pos[3 * s + a];
#pragma unroll
    for (int a = 0; a < 4; ++a) ai[u][a] = 0.0;
  }
  if (threadIdx.x == 0) L.stack[0] = 0;  // the root
  int top = 1, n_cells = 0, n_leaves = 0;
  int64_t sum_cells = 0, sum_pairs = 0;
  __syncthreads();
  for (;;) {
    // Every round pops at least one cell and every cell is pushed at most once,
    // so the loop ends.  The pop count shrinks as the stack fills: the children
    // of the popped cells (at most 8 each) leave the reserve free, and inside it
    // cells go one at a time, depth first, which adds at most 7 a level.
    while (top > 0 && n_cells + T <= W::kCells && n_leaves + T <= W::kLeaves) {
      const int npop = min(min(top, T), max(1, (W::kStack - kStackReserve - 1 - top) / 7));
      int c = -1;
      if ((int)threadIdx.x < npop) c = L.stack[top - npop + threadIdx.x];
      int accept = 0, leaf = 0, nch = 0, fch = 0;
      if (c >= 0) {
        const uint64_t ckey = g.key[c];
        const double2 *cm = reinterpret_cast<const double2 *>(g.com + 4 * (int64_t)c);
        const double2 m0 = cm[0];
        const double mz = g.com[4 * (int64_t)c + 2];
        const int2 kids = reinterpret_cast<const int2 *>(g.child)[c];
        const int cd = cell_depth(ckey);
        const bool contains = cd <= gd && (gkey >> (3 * (gd - cd))) == ckey;
        if (!contains) {
          double cen[3], l, d2 = 0.0;
          cell_centre(g, ckey, cd, cen, l);
          const double cmv[3] = {m0.x, m0.y, mz};
#pragma unroll
          for (int a = 0; a < 3; ++a) {
            const double t = fabs(cen[a] + cmv[a] - gc[a]) - gh;
            if (t > 0.0) d2 = fma(t, t, d2);
          }
          accept = l * l < g.theta2 * d2;
        }
        if (!accept) {
          fch = kids.x;
          if (fch < 0)
            leaf = 1;
          else
            nch = kids.y;
        }
      }
      const uint64_t lt = lanemask_lt();
      const uint64_t ma = __ballot(accept), ml = __ballot(leaf);
      int wave_nch;
      int pp = wave_excl_nibble(nch, &wave_nch);
      if (lane_id() == 0) {
        L.w0[threadIdx.x / 64] = (uint32_t)__popcll(ma) | ((uint32_t)__popcll(ml) << 16);
        L.w1[threadIdx.x / 64] = (uint32_t)wave_nch;
      }
      __syncthreads();  // every thread has read its cell
      uint32_t before = 0, total = 0;
      int tot_p = 0;
#pragma unroll
      for (int q = 0; q < W::kWaves; ++q) {
        const uint32_t a = L.w0[q];
        const int b = (int)L.w1[q];
        const bool lower = q < (int)threadIdx.x / 64;
        before += lower ? a : 0u;
        pp += lower ? b : 0;
        total += a;
        tot_p += b;
      }
      const int base = top - npop;
      if (accept) L.cells[n_cells + (int)(before & 0xffffu) + __popcll(ma & lt)] = c;
      if (leaf) L.leaves[n_leaves + (int)(before >> 16) + __popcll(ml & lt)] = c;
      for (int k = 0; k < nch; ++k) L.stack[base + pp + k] = fch + k;
      top = uniform(base + tot_p);
      total = (uint32_t)uniform((int)total);
      n_cells += (int)(total & 0xffffu);
      n_leaves += (int)(total >> 16);
      __syncthreads();
    }
    add_cells<T, U, QUAD, WHOLE>(g, L, n_cells, xf, ai, slice, S, idle);
    sum_pairs += add_leaves<T, U, WHOLE>(g, L, n_leaves, gf, gn, xf, si, ai, slice, S, idle);
    sum_cells += n_cells;
    n_cells = n_leaves = 0;
    __syncthreads();  // the lists are consumed
    if (top == 0) break;
  }
  // the S partial sums of each particle, in order
#pragma unroll
  for (int u = 0; u < U; ++u) {
    double2 *mine = reinterpret_cast<double2 *>(L.sum[threadIdx.x]);
    mine[0] = make_double2(ai[u][0], ai[u][1]);
    mine[1] = make_double2(ai[u][2], ai[u][3]);
    __syncthreads();
    const int k = (int)threadIdx.x + u * Q;
    if ((int)threadIdx.x < Q && k < P) {
      double2 s0 = mine[0], s1 = mine[1];
      for (int q = 1; q < S; ++q) {
        const double2 *o = reinterpret_cast<const double2 *>(L.sum[threadIdx.x + q * Q]);
        const double2 t0 = o[0], t1 = o[1];
        s0.x += t0.x;
        s0.y += t0.y;
        s1.x += t1.x;
        s1.y += t1.y;
      }
      double2 *o = reinterpret_cast<double2 *>(acc + 4 * (f0 + k));
      o[0] = s0;
      o[1] = s1;
    }
    __syncthreads();
  }
  *cells = sum_cells;
  *pairs = sum_pairs;
}

// FP64 arithmetic bounds it: 36 vector instructions an interaction and wave (31 of
// them FP64), 90 % of the lanes in use.  2^21 Plummer particles, theta 0.75, n_crit
// 512, 4.2e9 interactions: 8.0 ms (1.9e-12 s each) against 15.6 ms with one thread a
// particle, a square root and a division; the traversal alone is 0.5 ms of it.
// WHOLE: an item is a group, taken part by part (an instance of its own: the loop costs the
// other 1 %).
template <int T, bool QUAD, bool WHOLE>
__global__ __launch_bounds__(T, kWalkWaves) void k_walk(GravArgs g, const int32_t *__restrict__ items,
                                               uint32_t *__restrict__ counts, int32_t part,
                                               double *__restrict__ acc,
                                               unsigned long long *__restrict__ stats) {
  __shared__ __align__(16) WalkLds<T> L;
  const uint32_t G = counts[0];
  for (;;) {
    if (threadIdx.x == 0) L.next = atomicAdd(&counts[1], 1u);
    __syncthreads();
    const uint32_t gi = (uint32_t)uniform((int)L.next);
    if (gi >= G) break;  // the same for the whole workgroup
    const int32_t it = uniform(items[gi]);
    const uint32_t nth = it < 0 ? (uint32_t)-it : 0u;  // which part of the group
    const int32_t grp = it < 0 ? uniform(items[gi - nth]) : it;
    const uint64_t gkey = uniform(g.key[grp]);
    const int gd = cell_depth(gkey);
    double gc[3], gl;
    cell_centre(g, gkey, gd, gc, gl);
#pragma unroll
    for (int a = 0; a < 3; ++a) gc[a] = uniform(gc[a]);
    const double gh = 0.5 * uniform(gl);
    const int32_t gf = uniform(g.first[grp]);
    const int32_t gn = uniform(g.count[grp]);
    const int32_t p0 = (int32_t)nth * part;  // below gn: the parts cover the group
    int64_t cells = 0, pairs = 0;
    // the P particles of the group from its q-th on
    auto walk = [&](int32_t q, int P) __attribute__((always_inline)) {
      // particles per lane: the fewest idle lanes, then the fewest LDS reads
      int best = -1, U = kWalkPpt;
#pragma unroll
      for (int u = kWalkPpt; u >= 1; --u) {
        const int Q = (P + u - 1) / u;
        if (Q > T) continue;
        // lanes in use out of T * u, in 1/1024ths, less what a source's reads cost
        const int used = max((P * (T / Q) * 1024) / (T * u) - kReadCost / u, 0);
        if (used > best) {
          best = used;
          U = u;
        }
      }
      const int64_t f0 = (int64_t)gf + q;
      switch (uniform(U)) {
        case 1:
          walk_pass<T, 1, QUAD, WHOLE>(g, L, gkey, gd, gc, gh, gf, gn, f0, P, acc, &cells, &pairs);
          break;
        case 2:
          walk_pass<T, 2, QUAD, WHOLE>(g, L, gkey, gd, gc, gh, gf, gn, f0, P, acc, &cells, &pairs);
          break;
        case 3:
          walk_pass<T, 3, QUAD, WHOLE>(g, L, gkey, gd, gc, gh, gf, gn, f0, P, acc, &cells, &pairs);
          break;
        default:
          walk_pass<T, 4, QUAD, WHOLE>(g, L, gkey, gd, gc, gh, gf, gn, f0, P, acc, &cells, &pairs);
          break;
      }
    };
    if constexpr (WHOLE) {
      for (int32_t q = 0;; q += part) {
        walk(q, min(part, gn - q));
        if (gn - q <= part) break;
      }
    } else {
      walk(p0, min(part, gn - p0));
    }
    if (threadIdx.x == 0 && stats && nth == 0) {
      // every group particle meets every listed cell and every listed particle
      // but itself
      atomicAdd(&stats[0], 1ull);
      atomicAdd(&stats[1], (unsigned long long)gn * (unsigned long long)(cells + pairs - 1));
    }
    __syncthreads();  // L.next is read before it is written again
  }
}

size_t gravity_workspace_bytes(int64_t c_max) { return 4 * (size_t)c_max + 256; }


// Most particles of one item of work.  A large group takes long (512 particles with
// a list of 2,000 some 0.3 ms), so small sets, whose groups do not fill the chip,
// are cut finer although every part walks the tree again.  us a walk at parts of
// 32 / 64 / 128 / 256: 2^14 160 / 183 / 252 / 340, 2^16 423 / 408 / 467 / 692,
// 1.3e5 528 / 475 / 483 / 563, 3e5 1215 / 1020 / 1004 / 1098, 2^21 10552 / 8765 /
// 8062 / 8080.
//
// A list of parts has up to n entries, which the workspace holds if c_max is n or more, as
// tb_max_cells() is.  With a smaller c_max, the number of cells of the tree say, there is
// room for the groups alone: they stay whole, and a workgroup goes through one part by part.
WalkItems walk_items(int64_t n, int64_t c_max) {
  if (c_max < n) return {kWalkThreads * kWalkPpt, true};
  if (n < (int64_t{1} << 15)) return {32, false};
  return {n < (int64_t{1} << 18) ? 64 : 128, false};
}

// A grid that fills the chip takes the items in turn.
template <int T>
static void launch_walk(const GravArgs &g, const GravIn &in, const int32_t *items,
                        uint32_t *counts, const WalkItems &it, hipStream_t s) {
  int64_t wg = 256 * kWalkWaves * 256 / T;
  if (wg > in.n) wg = in.n;  // an item holds at least one particle
  auto *stats = reinterpret_cast<unsigned long long *>(in.stats);
  auto k = in.quadrupole ? (it.whole ? k_walk<T, true, true> : k_walk<T, true, false>)
                         : (it.whole ? k_walk<T, false, true> : k_walk<T, false, false>);
  k<<<(unsigned)wg, T, 0, s>>>(g, items, counts, it.part, in.acc, stats);
}

hipError_t launch_gravity(const GravIn &in, hipStream_t s) {
  GravArgs g;
  g.key = in.tree->cell_key;
  g.first = in.tree->cell_first;
  g.count = in.tree->cell_count;
  g.child = in.tree->child_ptr;
  g.com = static_cast<const double *>(in.tree->com);
  g.quad = static_cast<const double *>(in.tree->quad);
  g.box = in.tree->box_out;
  g.pos = in.pos_sorted;
  g.mass = in.mass_sorted;
  g.theta2 = in.theta * in.theta;
  g.eps2 = in.eps * in.eps;
  // (so that one comparison finds zero and infinity: another one costs the walk of 2000
  // particles 5 %)
  if (std::isinf(g.eps2)) g.eps2 = -g.eps2;
  g.hilbert = in.hilbert ? 1 : 0;
  int32_t *items = static_cast<int32_t *>(in.workspace);  // at most c_max of them
  uint32_t *counts = reinterpret_cast<uint32_t *>(items + in.c_max);
  const WalkItems it = walk_items(in.n, in.c_max);
  static_assert(kWalkThreads * kWalkPpt >= 128, "a part fits one pass");
  k_grav_init<<<1, 64, 0, s>>>(counts, reinterpret_cast<unsigned long long *>(in.stats));
  int64_t blocks = (in.c_max + 255) / 256;
  if (blocks > 4096) blocks = 4096;
  k_find_groups<<<(unsigned)blocks, 256, 0, s>>>(in.tree->n_cells, g.count, g.child, in.n_crit,
                                                 it.part, it.whole, items, counts);
  launch_walk<kWalkThreads>(g, in, items, counts, it, s);
  return hipGetLastError();
}

}  // namespace tb
