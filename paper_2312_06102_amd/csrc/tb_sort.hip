// tb_sort.hip -- stable LSD radix sort of (key, index) pairs (Sec. 2.3, step ii).
//
// One kernel launch per digit pass ("onesweep" structure):
//   * every workgroup takes the next tile of keys (dynamic tile id, so all
//     earlier tiles are already running and the look-back always progresses);
//   * each wave ranks its keys with 64-lane ballots: for every digit bit a
//     ballot, folded into the mask of lanes holding the same digit, whose
//     population below the lane is the lane's rank among equal digits; items
//     are processed in index order, so the ranking is stable;
//   * per-wave digit counts are combined in LDS; the tile publishes its
//     per-digit counts, then looks back over earlier tiles (decoupled look-back)
//     for its global exclusive prefix;
//   * keys and payloads are first sorted by digit inside the tile in LDS, then
//     written so that consecutive lanes store consecutive addresses of a digit
//     run.
// The global digit counts come from the key-generation pass (and become each
// digit's base once per build), so the keys are read only once per pass.
//
// The passes sort the upper 32 or 40 bits of the 63 (make_plan has the rule; all of them
// for n_leaf above 95).  The reorder orders the particles that agree in those by the rest
// of their keys and writes perm.  Passes over the low bits come first when the key
// kernel's sample has found that the keys crowd; they are launched in any case and return
// at once if not.
//
// By default the passes of a large single set are "counted" instead (reduce, then
// scan; a batch with TB_SORT_COUNTED too): a first kernel reads each element's
// digit (one byte, left behind by the previous pass or the key kernel) and
// writes every tile's digit counts, a second turns them into exclusive
// prefixes over the tiles, and the scatter kernel reads its tile's offsets
// instead of waiting on its predecessors.  Reading that byte again costs less
// than the look-back chain across the chip; TB_SORT_LOOKBACK keeps the
// look-back.
//
// A single set of up to 8192 particles is sorted by one workgroup in one launch
// (k_sort_one).
//
// A batch sorts every set in place: a set's tiles never straddle it, its tiles'
// look-back chain starts at its own first tile, and its digit runs start at
// bases taken from its own digit counts (counted per set by the key kernel).
// The passes thus give the (set, key) order with no pass over the set id.
//
// Elements shrink as the passes go: a pass carries only the key bits later passes
// still need.  The first reads the 64-bit key and writes it, without the bits that are
// consumed or not sorted, over the index in one packed word, (key bits << idx_bits) |
// index, whose digit is read at bit idx_bits; once both fit in 32 bits the word has 32.
// The last pass writes the index alone.  (The low passes move whole keys and indices in
// two arrays, and leave the upper bits packed where that fits.  Where every bit is sorted
// the first passes do the same, until the rest of the key fits beside the index.)  The
// sorted keys themselves are recomputed from the sorted particles in
// the reorder pass, which reads those particles anyway.
#include "tb_internal.h"

namespace tb {

template <int THREADS>
__device__ __forceinline__ uint32_t block_exclusive_sum(uint32_t v, uint32_t *s_tmp,
                                                        uint32_t *total) {
  constexpr int WAVES = THREADS / 64;
  const int wv = threadIdx.x / 64;
  const uint32_t inc = wave_inclusive_scan(v);
  if (lane_id() == 63) s_tmp[wv] = inc;
  __syncthreads();
  uint32_t off = 0, tot = 0;
#pragma unroll
  for (int k = 0; k < WAVES; ++k) {
    const uint32_t t = s_tmp[k];
    off += (k < wv) ? t : 0u;
    tot += t;
  }
  __syncthreads();
  *total = tot;
  return off + inc - v;
}

// Word type of an element format (kFormIdx and kFormPack32: 32-bit words).
template <int F>
struct FormType {
  using T = uint32_t;
};
template <>
struct FormType<kFormKey64> {
  using T = uint64_t;
};
template <>
struct FormType<kFormPack64> {
  using T = uint64_t;
};
template <>
struct FormType<kFormLow> {
  using T = uint64_t;
};

// Digit at bit offset `shift` (uniform): the pass's digit position for a 64-bit
// key, idx_bits for a packed element.
template <int BITS>
__device__ __forceinline__ uint32_t digit_of(uint64_t k, int shift) {
  const uint32_t lo = (uint32_t)k, hi = (uint32_t)(k >> 32);
  const uint32_t w = shift < 32 ? __builtin_amdgcn_alignbit(hi, lo, (uint32_t)shift)
                                : (hi >> (shift - 32));
  return w & ((1u << BITS) - 1u);
}
template <int BITS>
__device__ __forceinline__ uint32_t digit_of(uint32_t k, int shift) {
  return (k >> shift) & ((1u << BITS) - 1u);
}

// Tiles of a pass.  A single set: tile t holds keys [t TILE, (t+1) TILE) of the
// array, and the digit runs start where the global digit counts put them.  A
// batch: every set is sorted in place; a set's tiles never straddle it, tile t
// of set b holds the set's keys [t TILE, (t+1) TILE) counted from the set's
// first tile, and each digit's run of the set starts at the set's own base.
struct SegTiles {
  const int64_t *tile_start;  // [B + 1] first tile of each set, or NULL (single set)
  const int32_t *tile_set;    // [tiles] set of each tile
  const int64_t *set_off;     // [B + 1] first position of each set
  size_t base_stride;         // words between two sets' rows of `hist`
  int32_t nsets;
};

// Digit counts of the tiles of a counted pass: tile t (its elements as the
// scatter kernel tiles them, SegTiles) gets cnt[d][t].  The digits come from
// dig, written for this pass by the key kernel (first pass) or by the previous
// pass's scatter, so a count reads one byte an element (two for 9-bit digits)
// instead of the element.  A workgroup counts TPW consecutive tiles at once
// (every thread's loads of all of them in flight together, one set of per-wave
// histograms per tile), which halves the waves for about the same wave life.
template <int BITS, int IPT, int THREADS, int TPW>
__global__ __launch_bounds__(THREADS) void k_tile_count(const void *__restrict__ dig_v, uint32_t n,
                                                        uint32_t *__restrict__ cnt,
                                                        uint32_t n_tiles, SegTiles seg) {
  using DT = DigitType<BITS>;
  constexpr int R = 1 << BITS;
  constexpr int WAVES = THREADS / 64;
  constexpr uint32_t TILE = (uint32_t)THREADS * IPT;
  __shared__ uint32_t h[TPW * WAVES * R];  // per tile, one histogram per wave
  for (int i = threadIdx.x; i < TPW * WAVES * R; i += THREADS) h[i] = 0;
  const DT *__restrict__ dig = static_cast<const DT *>(dig_v);
  const uint32_t t0 = blockIdx.x * TPW;
  const uint32_t tiles_here = seg.tile_start ? (uint32_t)seg.tile_start[seg.nsets] : n_tiles;
  uint32_t base[TPW], last[TPW];
#pragma unroll
  for (int q = 0; q < TPW; ++q) {
    const uint32_t tile = t0 + q;
    base[q] = tile * TILE;
    uint32_t hi = n;
    if (tile >= tiles_here) {  // past the last tile: counts nothing
      base[q] = 1u;
      hi = 1u;
    } else if (seg.tile_start) {
      const int b = seg.tile_set[tile];
      base[q] = (uint32_t)seg.set_off[b] + (uint32_t)((int64_t)(tile - seg.tile_start[b]) * TILE);
      hi = (uint32_t)seg.set_off[b + 1];
    }
    last[q] = min(base[q] + TILE, hi) - 1u;  // base[q] - 1 when the tile is empty
  }
  uint32_t k[TPW][IPT];
#pragma unroll
  for (int q = 0; q < TPW; ++q)
#pragma unroll
    for (int j = 0; j < IPT; ++j)
      k[q][j] = dig[min(min(base[q] + j * THREADS + threadIdx.x, last[q]), n - 1u)];
  __syncthreads();
#pragma unroll
  for (int q = 0; q < TPW; ++q) {
    uint32_t *hw = h + (q * WAVES + threadIdx.x / 64) * R;
#pragma unroll
    for (int j = 0; j < IPT; ++j) {
      const bool valid = base[q] + j * THREADS + threadIdx.x <= last[q] &&
                         base[q] <= last[q];
      const uint32_t d = k[q][j];
      // clustered data gives few distinct digits per wave: groups of four or
      // more equal digits add once (all masks wave-uniform), the rest one by one
      uint64_t rem = __ballot(valid);
      while (rem != 0) {
        const int l = __builtin_ctzll(rem);
        const uint32_t d0 = __builtin_amdgcn_readlane(d, l);
        const uint64_t m = __ballot(d == d0) & rem;
        const uint32_t c = (uint32_t)__popcll(m);
        if (c < 4) break;
        if (lane_id() == l) atomicAdd(&hw[d0], c);
        rem &= ~m;
      }
      if ((rem >> lane_id()) & 1u) atomicAdd(&hw[d], 1u);
    }
  }
  __syncthreads();
  for (int i = threadIdx.x; i < TPW * R; i += THREADS) {
    const int q = i / R, d = i % R;
    if (t0 + q >= tiles_here) continue;
    uint32_t c = 0;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) c += h[(q * WAVES + w) * R + d];
    cnt[(size_t)d * n_tiles + t0 + q] = c;
  }
}

// cnt[d][t] <- sum over t' < t of cnt[d][t']: one workgroup per digit, each
// thread a contiguous run of tiles.
template <int THREADS>
__global__ __launch_bounds__(THREADS) void k_tile_scan(uint32_t *__restrict__ cnt,
                                                       uint32_t n_tiles) {
  __shared__ uint32_t s_tmp[THREADS / 64];
  uint32_t *row = cnt + (size_t)blockIdx.x * n_tiles;
  const uint32_t per = (n_tiles + THREADS - 1) / THREADS;
  const uint32_t t0 = min(threadIdx.x * per, n_tiles), t1 = min(t0 + per, n_tiles);
  uint32_t sum = 0;
  for (uint32_t t = t0; t < t1; ++t) sum += row[t];
  uint32_t total;
  uint32_t run = block_exclusive_sum<THREADS>(sum, s_tmp, &total);
  for (uint32_t t = t0; t < t1; ++t) {
    const uint32_t c = row[t];
    row[t] = run;
    run += c;
  }
}


// All ones if bit b of d is set, else zero: one signed one-bit field extract
// (the compiler would otherwise shift left and then arithmetically right).
__device__ __forceinline__ uint32_t lane_bit_mask(uint32_t d, int b) {
  uint32_t m;
  asm("v_bfe_i32 %0, %1, %2, 1" : "=v"(m) : "v"(d), "i"(b));
  return m;
}

// Shape and LDS of one radix tile.  FIN / FOUT: element format read / written
// (FIN is never kFormIdx, FOUT never kFormLow).
template <int BITS, int IPT, int THREADS, int FIN, int FOUT>
struct Sweep {
  using KI = typename FormType<FIN>::T;
  using KO = typename FormType<FOUT>::T;
  // packed input: the index is in the word
  static constexpr bool PIN = FIN != kFormKey64 && FIN != kFormLow;
  static constexpr int R = 1 << BITS;
  static constexpr int WAVES = THREADS / 64;
  static constexpr int TILE = THREADS * IPT;
  static constexpr int DPT = (R + THREADS - 1) / THREADS;  // digits per thread
  // the local sort keeps the input word, except where only a separate index is
  // written: there the digit of each slot suffices
  static constexpr bool SLOT_DIGIT = FOUT == kFormIdx && !PIN;
  static constexpr int SLOT_BYTES = SLOT_DIGIT ? 2 : (int)sizeof(KI);
  struct Lds {
    alignas(16) unsigned char slot[TILE * SLOT_BYTES];
    uint32_t vals[PIN ? 1 : TILE];
    uint32_t wc[WAVES * R];   // per-wave digit counters, then wave offsets
    uint32_t tstart[R];       // tile-local start of each digit
    int32_t goff[R];          // output position minus tile-local position
    uint32_t tmp[WAVES];
    uint32_t tile;
  };
};

// Wave-striped load of a tile: item j of lane l is element wbase + j*64, with
// wbase = lo + wave*64*IPT + l.  Loads are branch-free (indices past the tile
// are clamped and the items masked later) so that all of them are in flight
// together.  v: the separate index of kFormKey64; when vin is NULL, the position
// less vbase (the set's first position in a batch, whose sort carries indices
// within the set).  in_word > 0: the words are key bits above an index of that many bits
// all the same; the key bits then move up by `shift`.
template <class S, int IPT>
__device__ __forceinline__ void sweep_load(const typename S::KI *__restrict__ kin,
                                           const uint32_t *__restrict__ vin, uint32_t wbase,
                                           uint32_t last, uint32_t vbase,
                                           typename S::KI (&k)[IPT], uint32_t (&v)[IPT],
                                           int in_word = 0, int shift = 0) {
#pragma unroll
  for (int j = 0; j < IPT; ++j) k[j] = kin[min(wbase + j * 64, last)];
  if constexpr (!S::PIN) {
    if (in_word > 0) {
#pragma unroll
      for (int j = 0; j < IPT; ++j) {
        v[j] = (uint32_t)k[j] & (in_word >= 32 ? 0xffffffffu : (1u << in_word) - 1u);
        k[j] = (k[j] >> in_word) << shift;
      }
    } else if (vin) {
#pragma unroll
      for (int j = 0; j < IPT; ++j) v[j] = vin[min(wbase + j * 64, last)];
    } else {
#pragma unroll
      for (int j = 0; j < IPT; ++j) v[j] = wbase + j * 64 - vbase;
    }
  }
}

// Ranks a loaded tile and sorts it by digit in LDS.  On entry L.wc is zero
// (behind a barrier).  On return, for each digit d = threadIdx.x * DPT + t:
// tcnt[t] its count in the tile and trun[t] its tile-local start; with PUBLISH
// the tile's per-digit counts are also published for the look-back (inclusive
// when it is the first tile of its set).
template <class S, int BITS, int IPT, int THREADS, bool PUBLISH>
__device__ __forceinline__ void sweep_rank(typename S::Lds &L, const typename S::KI (&k)[IPT],
                                           const uint32_t (&v)[IPT], uint32_t wbase,
                                           uint32_t last, int shift, uint64_t *status,
                                           uint32_t tile, bool first, uint32_t (&tcnt)[S::DPT],
                                           uint32_t (&trun_d)[S::DPT]) {
  constexpr int R = S::R, WAVES = S::WAVES, DPT = S::DPT;
  const int wv = threadIdx.x / 64;
  const uint64_t lt = lanemask_lt();
  uint32_t dg[IPT], rk[IPT];
#pragma unroll
  for (int j = 0; j < IPT; ++j) dg[j] = digit_of<BITS>(k[j], shift);

  // Stable wave-level ranking: for every digit bit a ballot; XNOR-ing the
  // ballot with "all ones if my bit is set" keeps exactly the lanes that agree
  // with me on that bit, so the AND over all bits is the set of lanes holding
  // my digit.  Its population below my lane is my rank among them.  (The mask
  // is a signed one-bit field extract, which also feeds the ballot, and each
  // half of the AND is one three-input bit operation: four instructions a bit.
  // The operation's table is indexed by (a, b, c) bits as a*4 + b*2 + c, so
  // a & ~(b ^ c) is 0xF0 & ~(0xCC ^ 0xAA) = 0x90.)
  uint32_t *wc = L.wc + wv * R;
#pragma unroll
  for (int j = 0; j < IPT; ++j) {
    const bool valid = wbase + j * 64 <= last;
    const uint32_t d = dg[j];
    const uint64_t vmask = __ballot(valid);
    uint32_t plo = (uint32_t)vmask, phi = (uint32_t)(vmask >> 32);
#pragma unroll
    for (int b = 0; b < BITS; ++b) {
      const uint32_t m = lane_bit_mask(d, b);  // bit b set: all ones
      const uint64_t bb = __ballot(m != 0u);
      plo = __builtin_amdgcn_bitop3_b32(plo, (uint32_t)bb, m, 0x90);
      phi = __builtin_amdgcn_bitop3_b32(phi, (uint32_t)(bb >> 32), m, 0x90);
    }
    const uint64_t peers = ((uint64_t)phi << 32) | plo;
    const uint32_t pre = (uint32_t)__popcll(peers & lt);
    uint32_t cnt = 0;
    if (valid) cnt = wc[d];
    rk[j] = cnt + pre;
    if (valid && pre == 0) wc[d] = cnt + (uint32_t)__popcll(peers);
  }
  __syncthreads();

  // per digit: exclusive offsets across waves and the tile count
#pragma unroll
  for (int t = 0; t < DPT; ++t) {
    const int d = threadIdx.x * DPT + t;
    uint32_t run = 0;
    if (d < R) {
#pragma unroll
      for (int q = 0; q < WAVES; ++q) {
        const uint32_t c = L.wc[q * R + d];
        L.wc[q * R + d] = run;
        run += c;
      }
      if constexpr (PUBLISH)
        atomic_store_agent(&status[(size_t)tile * R + d],
                           (first ? kFlagInclusive : kFlagAggregate) | (uint64_t)run);
    }
    tcnt[t] = run;
  }

  // tile-local digit starts: a block scan over the digits
  uint32_t tsum = 0;
#pragma unroll
  for (int t = 0; t < DPT; ++t) tsum += tcnt[t];
  uint32_t dummy;
  uint32_t trun = block_exclusive_sum<THREADS>(tsum, L.tmp, &dummy);
#pragma unroll
  for (int t = 0; t < DPT; ++t) {
    const int d = threadIdx.x * DPT + t;
    if (d < R) L.tstart[d] = trun;
    trun_d[t] = trun;
    trun += tcnt[t];
  }
  __syncthreads();

  // sort the tile by digit in LDS (the input word, or the digit where only a
  // separate index is written)
#pragma unroll
  for (int j = 0; j < IPT; ++j) {
    if (wbase + j * 64 <= last) {
      const uint32_t d = dg[j];
      const uint32_t p = L.tstart[d] + wc[d] + rk[j];
      if constexpr (S::SLOT_DIGIT)
        reinterpret_cast<uint16_t *>(L.slot)[p] = (uint16_t)d;
      else
        reinterpret_cast<typename S::KI *>(L.slot)[p] = k[j];
      if constexpr (!S::PIN) L.vals[p] = v[j];
    }
  }
}

// Coalesced scatter of a tile sorted in LDS (L.goff set, behind a barrier):
// consecutive lanes write consecutive slots of a digit run, inside [set_lo, hi).
// A packed output word holds the key bits above this digit over the index; the
// last pass writes the index plus set_lo (a batch's indices are within the set).
// dig_out (a counted next pass): the next pass's digit of each element, at its
// output position.
template <class S, int BITS, int THREADS, int FOUT>
__device__ __forceinline__ void sweep_scatter(const typename S::Lds &L, uint32_t tile_n, int shift,
                                              int ib, uint32_t set_lo, uint32_t hi,
                                              typename S::KO *__restrict__ kout,
                                              uint32_t *__restrict__ vout,
                                              DigitType<BITS> *__restrict__ dig_out, bool &bad) {
  using KI = typename S::KI;
  using KO = typename S::KO;
  const uint32_t idx_mask = ib >= 32 ? 0xffffffffu : (1u << ib) - 1u;
  for (uint32_t i = threadIdx.x; i < tile_n; i += THREADS) {
    uint32_t d;
    KI kk = 0;
    if constexpr (S::SLOT_DIGIT) {
      d = reinterpret_cast<const uint16_t *>(L.slot)[i];
    } else {
      kk = reinterpret_cast<const KI *>(L.slot)[i];
      d = digit_of<BITS>(kk, shift);
    }
    const uint32_t idx = S::PIN ? ((uint32_t)kk & idx_mask) : L.vals[i];
    const uint32_t gp = (uint32_t)(L.goff[d] + (int32_t)i);
    if (gp < set_lo || gp >= hi) {  // cannot happen with consistent digit counts
      bad = true;
      continue;
    }
    if constexpr (FOUT == kFormIdx) {
      vout[gp] = idx + set_lo;
    } else {
      // the key bits above this digit: the next pass's digit at their bottom
      const uint64_t rest = (uint64_t)kk >> (shift + BITS);
      if constexpr (FOUT == kFormKey64) {
        kout[gp] = (KO)kk;
        vout[gp] = idx;
      } else {
        kout[gp] = (KO)((rest << ib) | idx);
      }
      if (dig_out) dig_out[gp] = (DigitType<BITS>)(rest & ((1u << BITS) - 1u));
    }
  }
}

// One radix pass, one workgroup per tile.  kin/kout hold the key or packed
// words; vin/vout the separate index of kFormKey64 (vin NULL: the index is the
// position) and the output of kFormIdx.  shift: the digit's bit offset in the
// input word; ib: idx_bits; key_mask: the bits of a whole key that a packed word keeps.
// hist: the pass's digit bases, where each digit's
// run starts in the output [radix]; a batch has a row per set (set b at b *
// base_stride).
//
// Waves a SIMD a pass's registers must allow (the second launch bound; 1: no
// limit).  With 8-bit digits a pass over 32-bit packed words needs little LDS,
// so held to six waves (80 VGPRs, a 12-byte spill a lane) it runs three
// 512-thread workgroups a CU instead of two: 47.6 -> 43.8 us at 2^24.  So does
// a batch's look-back pass over 64-bit packed words with 5120-key tiles (a
// 28-byte spill; the 4096-set batch's sort 6.45 -> 6.34 ms), while the counted
// single-set pass loses more to its spill than it gains (sort 0.79 -> 0.87 ms)
// and larger tiles leave no LDS for a third workgroup.
// The conditional passes' loop over tiles is held to four waves (two workgroups a CU)
// where the LDS of two fits.
template <int BITS, int IPT, int THREADS, int FIN, int FOUT, bool COUNTED, bool SEG>
constexpr int sweep_waves() {
  if (FIN == kFormLow) return THREADS == 512 && IPT <= 11 ? 4 : 1;
  if (BITS != 8) return 1;
  if (FIN == kFormPack32) return 6;
  if (FIN == kFormPack64 && SEG && !COUNTED && THREADS == 512 && THREADS * IPT <= 5120) return 6;
  return 1;
}

// One tile of a pass; false when the pass has no more.
template <int BITS, int IPT, int THREADS, int FIN, int FOUT, bool COUNTED, bool SEG>
__device__ __forceinline__ bool sweep_tile(
    typename Sweep<BITS, IPT, THREADS, FIN, FOUT>::Lds &L, const void *__restrict__ kin_v,
    void *__restrict__ kout_v, const uint32_t *__restrict__ vin, uint32_t *__restrict__ vout,
    uint32_t n, int shift, int ib, uint64_t key_mask, const uint32_t *__restrict__ hist,
    uint64_t *__restrict__ status, uint64_t *__restrict__ status_next,
    uint32_t *__restrict__ tile_counter, const uint32_t *__restrict__ tile_off,
    int32_t *__restrict__ status_word, uint32_t n_tiles, const SegTiles &seg,
    void *__restrict__ dig_out, int in_word) {
  using S = Sweep<BITS, IPT, THREADS, FIN, FOUT>;
  using KI = typename S::KI;
  constexpr int R = S::R, WAVES = S::WAVES, TILE = S::TILE, DPT = S::DPT;
  constexpr bool LOW = FIN == kFormLow;
  const KI *__restrict__ kin = static_cast<const KI *>(kin_v);
  typename S::KO *__restrict__ kout = static_cast<typename S::KO *>(kout_v);
  constexpr bool batch = SEG;

  // Look-back passes take tiles in the order they start, so that every earlier
  // tile is already running; counted passes need no order.  The conditional passes'
  // workgroups take tile after tile.
  if (!COUNTED && threadIdx.x == 0) L.tile = atomicAdd(tile_counter, 1u);
  for (int i = threadIdx.x; i < WAVES * R; i += THREADS) L.wc[i] = 0;
  __syncthreads();
  const uint32_t tile = COUNTED ? xcd_tile(blockIdx.x, gridDim.x) : L.tile;
  // a batch launches one workgroup for each tile it may have
  const uint32_t tiles_here = batch ? (uint32_t)seg.tile_start[seg.nsets] : n_tiles;
  if (tile >= tiles_here) {
    // a single set launches one workgroup per tile: the counter was not reset
    if (!LOW && !batch && threadIdx.x == 0) atomicOr(status_word, TB_STATUS_INTERNAL);
    return false;
  }
  // the tile's elements [lo, lo + tile_n); its set's first tile starts the look-back
  uint32_t lo = tile * (uint32_t)TILE, hi = n, set_lo = 0u, set_tile0 = 0u;
  bool first = tile == 0;
  const uint32_t *digit_base = hist;
  if constexpr (batch) {
    const int b = seg.tile_set[tile];
    const int64_t t0 = seg.tile_start[b];
    set_tile0 = (uint32_t)t0;
    set_lo = (uint32_t)seg.set_off[b];
    lo = set_lo + (uint32_t)((int64_t)(tile - t0) * TILE);
    hi = (uint32_t)seg.set_off[b + 1];
    first = (int64_t)tile == t0;
    digit_base = hist + (size_t)b * seg.base_stride;
  }
  const uint32_t tile_n = (hi - lo) < (uint32_t)TILE ? (hi - lo) : (uint32_t)TILE;
  const uint32_t last = lo + tile_n - 1u;
  // where each digit's run starts does not depend on the elements: load it first
  uint32_t g[DPT];
#pragma unroll
  for (int t = 0; t < DPT; ++t) {
    const int d = threadIdx.x * DPT + t;
    g[t] = (d < R) ? digit_base[d] : 0u;
  }
  const uint32_t wbase = lo + (uint32_t)(threadIdx.x / 64) * 64u * IPT + (uint32_t)lane_id();
  KI k[IPT];
  uint32_t v[IPT];
  sweep_load<S, IPT>(kin, vin, wbase, last, set_lo, k, v, in_word, shift);
  if constexpr (!S::PIN && FOUT != kFormKey64) {
#pragma unroll
    for (int j = 0; j < IPT; ++j) k[j] &= key_mask;
  }

  uint32_t tcnt[DPT], trun_d[DPT];
  sweep_rank<S, BITS, IPT, THREADS, !COUNTED>(L, k, v, wbase, last, shift, status, tile, first,
                                               tcnt, trun_d);
  // where each digit's run starts in the output: g, the pass's digit bases
  // the next pass's look-back words for this tile start cleared
  for (int i = threadIdx.x; i < R; i += THREADS) status_next[(size_t)tile * R + i] = 0;

  // the counted offsets (or the decoupled look-back within the set), one thread per digit
#pragma unroll
  for (int t = 0; t < DPT; ++t) {
    const int d = threadIdx.x * DPT + t;
    if (d < R) {
      uint32_t excl = 0;
      if (COUNTED) {
        // the prefix over all earlier tiles, less the prefix before the set's first tile
        excl = tile_off[(size_t)d * n_tiles + tile];
        if (batch) excl -= tile_off[(size_t)d * n_tiles + set_tile0];
      } else if (!first) {
        bool timed_out = false;
        excl = lookback<2>(status, R, tile, d, timed_out);
        if (timed_out) atomicOr(status_word, TB_STATUS_INTERNAL);
        atomic_store_agent(&status[(size_t)tile * R + d],
                           kFlagInclusive | (uint64_t)(excl + tcnt[t]));
      }
      L.goff[d] = (int32_t)(g[t] + excl - trun_d[t]);
    }
  }
  __syncthreads();

  bool bad = false;
  sweep_scatter<S, BITS, THREADS, FOUT>(L, tile_n, shift, ib, set_lo, hi, kout, vout,
                                        static_cast<DigitType<BITS> *>(dig_out), bad);
  if (__ballot(bad) != 0 && lane_id() == 0) atomicOr(status_word, TB_STATUS_INTERNAL);
  return true;
}

template <int BITS, int IPT, int THREADS, int FIN, int FOUT, bool COUNTED, bool SEG>
__global__ __launch_bounds__(THREADS, (sweep_waves<BITS, IPT, THREADS, FIN, FOUT, COUNTED, SEG>())) void k_onesweep(
    const void *__restrict__ kin, void *__restrict__ kout, const uint32_t *__restrict__ vin,
    uint32_t *__restrict__ vout, uint32_t n, int shift, int ib, uint64_t key_mask,
    const uint32_t *__restrict__ hist,
    uint64_t *__restrict__ status, uint64_t *__restrict__ status_next,
    uint32_t *__restrict__ tile_counter, const uint32_t *__restrict__ tile_off,
    int32_t *__restrict__ status_word, uint32_t n_tiles, SegTiles seg, void *__restrict__ dig_out,
    const uint32_t *__restrict__ full, int low_word) {
  __shared__ typename Sweep<BITS, IPT, THREADS, FIN, FOUT>::Lds L;
  // The conditional passes sort the low bits, if the sample asked for it; the first pass
  // over the upper bits takes their order and words (low_word) then, else the input's.
  // (Where every bit is sorted in any case, the sample always asks.)
  constexpr bool LOW = FIN == kFormLow;
  int in_word = 0;
  if constexpr (FIN == kFormKey64 || LOW) {
    if (*full == 0u) {
      if constexpr (LOW) return;
      vin = nullptr;
    } else if (!LOW) {
      in_word = low_word;
    }
  }
  if constexpr (LOW) {
    while (sweep_tile<BITS, IPT, THREADS, FIN, FOUT, COUNTED, SEG>(
        L, kin, kout, vin, vout, n, shift, ib, key_mask, hist, status, status_next, tile_counter,
        tile_off, status_word, n_tiles, seg, dig_out, in_word))
      __syncthreads();  // the tile's LDS is read out
  } else {
    sweep_tile<BITS, IPT, THREADS, FIN, FOUT, COUNTED, SEG>(
        L, kin, kout, vin, vout, n, shift, ib, key_mask, hist, status, status_next, tile_counter,
        tile_off, status_word, n_tiles, seg, dig_out, in_word);
  }
}

// One launch of a pass: pass p.key_passes + k is the conditional low pass k.
template <int BITS, int IPT, int THREADS, int FIN, int FOUT, bool COUNTED>
static hipError_t launch_sweep(const Plan &p, const Work &w, int pass, const void *kin, void *kout,
                               const uint32_t *vin, uint32_t *vout, int shift, uint64_t *status,
                               uint64_t *status_next, void *dig_out, const tb_tree &out,
                               hipStream_t s) {
  const int R = 1 << BITS;
  SegTiles seg{nullptr, nullptr, nullptr, 0, p.nsets};
  const uint32_t *hist = w.hist + (size_t)pass * R;
  if (p.seg) {
    seg = SegTiles{w.seg_tile_start, w.seg_tile_set, w.set_off,
                   (size_t)(p.key_passes + p.low_passes) * R, p.nsets};
    hist = w.seg_base + (size_t)pass * R;
  }
  if constexpr (COUNTED) {
    constexpr int TPW = 2;
    k_tile_count<BITS, IPT, THREADS, TPW>
        <<<(unsigned)((p.sort_tiles + TPW - 1) / TPW), THREADS, 0, s>>>(
            w.dig, (uint32_t)p.n, w.tile_off, (uint32_t)p.sort_tiles, seg);
    // tiles past the batch's last one count nothing and come after every real
    // tile, so the scan's prefixes for the real tiles are unaffected
    k_tile_scan<1024><<<R, 1024, 0, s>>>(w.tile_off, (uint32_t)p.sort_tiles);
  }
  auto k = p.seg ? k_onesweep<BITS, IPT, THREADS, FIN, FOUT, COUNTED, true>
                 : k_onesweep<BITS, IPT, THREADS, FIN, FOUT, COUNTED, false>;
  // (a small grid of the conditional passes returns sooner when there is nothing to do;
  // at 2^26 6.8 us with a workgroup a tile, 3.8 us so)
  constexpr bool kLow = FIN == kFormLow;
  const uint64_t key_mask = p.skip_bits > 0 ? ~(1ull << 63) : ~0ull;
  const int64_t grid = kLow && p.sort_tiles > 512 ? 512 : p.sort_tiles;
  k<<<(unsigned)grid, THREADS, 0, s>>>(
      kin, kout, vin, vout, (uint32_t)p.n, shift, p.idx_bits, key_mask, hist, status, status_next,
      w.counters + pass, w.tile_off, out.status, (uint32_t)p.sort_tiles, seg, dig_out,
      w.counters + kFullSortCounter, pass == 0 && p.low_packed ? p.idx_bits : 0);
  return hipGetLastError();
}

template <int BITS, int IPT, int THREADS, int FIN, int FOUT>
static hipError_t launch_pass_c(const Plan &p, const Work &w, int pass, const tb_tree &out,
                                hipStream_t s) {
  const int P = p.key_passes;
  void *K[2] = {w.keys0, w.keys1};
  uint64_t *S[2] = {w.status0, w.status1};
  const int shift = FIN == kFormKey64 ? p.skip_bits + pass * BITS : p.idx_bits;
  // a counted pass that follows needs this pass to leave its digits behind
  void *dig_out = (pass + 1 < P && ((p.counted >> (pass + 1)) & 1u)) ? w.dig : nullptr;
  auto go = ((p.counted >> pass) & 1u) ? launch_sweep<BITS, IPT, THREADS, FIN, FOUT, true>
                                       : launch_sweep<BITS, IPT, THREADS, FIN, FOUT, false>;
  // the indices beside whole keys: the low passes' in the first pass, by turns in two arrays
  // where every bit is sorted (the first pass then starts from the positions)
  uint32_t *V[2] = {reinterpret_cast<uint32_t *>(out.perm), w.vals1};
  const uint32_t *vin = pass == 0 && p.skip_bits == 0 ? nullptr : V[(pass + 1) % 2];
  uint32_t *vout = FOUT == kFormIdx ? sorted_order(p, w, out) : V[pass % 2];
  return go(p, w, pass, K[pass % 2], K[(pass + 1) % 2], vin, vout, shift, S[pass % 2],
            S[(pass + 1) % 2], dig_out, out, s);
}

// The format pairs make_plan produces for 8- and 9-bit digits and any N below 2^31.
#define TB_SORT_PAIRS(PAIR)                                                               \
  PAIR(kFormKey64, kFormKey64) PAIR(kFormKey64, kFormPack64) PAIR(kFormPack64, kFormPack64) \
  PAIR(kFormPack64, kFormPack32) PAIR(kFormPack64, kFormIdx) PAIR(kFormPack32, kFormPack32) \
  PAIR(kFormPack32, kFormIdx)

bool sort_pair_built(int form_in, int form_out) {
#define TB_PAIR(FI, FO) \
  if (form_in == FI && form_out == FO) return true;
  TB_SORT_PAIRS(TB_PAIR)
#undef TB_PAIR
  return false;
}

template <int BITS, int IPT, int THREADS>
static hipError_t launch_pass_t(const Plan &p, const Work &w, int pass, const tb_tree &out,
                                hipStream_t s) {
  const int fi = p.form[pass], fo = p.form[pass + 1];
#define TB_PAIR(FI, FO) \
  if (fi == FI && fo == FO) return launch_pass_c<BITS, IPT, THREADS, FI, FO>(p, w, pass, out, s);
  TB_SORT_PAIRS(TB_PAIR)
#undef TB_PAIR
  return hipErrorInvalidValue;
}

// The conditional passes over the low key bits, before the others: whole keys and
// their indices from keys0 through the space of the sorted records and back to keys0,
// the indices through perm and vals1 to vals1 (or, once both fit a word, the upper bits
// packed above the index to keys0).  They look back whatever the others do
// (their launches return at once unless the sample asked for them), on the look-back
// words that leave status0 clear for the first pass that follows.
template <int BITS, int IPT, int THREADS>
static hipError_t launch_low_t(const Plan &p, const Work &w, const tb_tree &out, hipStream_t s) {
  const int L = p.low_passes;
  uint64_t *A = reinterpret_cast<uint64_t *>(w.sorted);
  uint64_t *K[2] = {A, A + p.n};
  uint32_t *V[2] = {w.vals1, reinterpret_cast<uint32_t *>(out.perm)};
  uint64_t *S[2] = {w.status0, w.status1};
  const uint64_t *kin = w.keys0;
  const uint32_t *vin = nullptr;
  for (int k = 0; k < L; ++k) {
    const bool last = k + 1 == L;
    uint64_t *kout = last ? w.keys0 : K[k % 2];
    uint32_t *vout = V[(L - 1 - k) % 2];
    void *dig_out = last && (p.counted & 1u) ? w.dig : nullptr;
    auto go = last && p.low_packed
                  ? launch_sweep<BITS, IPT, THREADS, kFormLow, kFormPack64, false>
                  : launch_sweep<BITS, IPT, THREADS, kFormLow, kFormKey64, false>;
    const hipError_t e = go(p, w, p.key_passes + k, kin, kout, vin, vout, low_shift(p, k),
                            S[(k + L) % 2], S[(k + L + 1) % 2], dig_out, out, s);
    if (e != hipSuccess) return e;
    kin = kout;
    vin = vout;
  }
  return hipSuccess;
}

// A single set that fits one tile: every pass in one launch of one workgroup, the words and
// their indices in LDS in between.  After the upper bits' passes the workgroup looks for
// runs longer than the reorder finishes and, if there is one (or the reorder finishes
// none), sorts by all key bits instead: then *full is set.  So neither the digit counts
// nor the conditional passes nor k_sort_runs are launched, 11 launches fewer: builds of
// 1000 Plummer particles 82 -> 58 us, 4096 93 -> 74, 8192 97 -> 86.  The next power of two
// would not fit the LDS of a CU.
constexpr int kOneThreads = 1024;

template <int IPT>
__global__ __launch_bounds__(kOneThreads) void k_sort_one(const uint64_t *__restrict__ keys,
                                                          uint32_t *__restrict__ order,
                                                          uint32_t n, int skip, int all,
                                                          uint32_t *__restrict__ full) {
  using S = Sweep<8, IPT, kOneThreads, kFormKey64, kFormKey64>;
  __shared__ typename S::Lds L;
  const uint32_t last = n - 1u;
  const uint32_t wbase = (threadIdx.x / 64) * 64u * IPT + (uint32_t)lane_id();
  uint64_t *slot = reinterpret_cast<uint64_t *>(L.slot);
  auto sort_from = [&](int from) {
    uint64_t k[IPT];
    uint32_t v[IPT], tcnt[S::DPT], trun[S::DPT];
    sweep_load<S, IPT>(keys, nullptr, wbase, last, 0u, k, v);
    for (int shift = from; shift < 63; shift += 8) {
      if (shift != from) {
#pragma unroll
        for (int j = 0; j < IPT; ++j) {
          const uint32_t x = min(wbase + j * 64, last);
          k[j] = slot[x];
          v[j] = L.vals[x];
        }
      }
      for (int i = threadIdx.x; i < S::WAVES * S::R; i += kOneThreads) L.wc[i] = 0;
      __syncthreads();
      sweep_rank<S, 8, IPT, kOneThreads, false>(L, k, v, wbase, last, shift, nullptr, 0u, true,
                                                tcnt, trun);
      __syncthreads();
    }
  };
  bool every_bit = all != 0;
  if (!every_bit) {
    sort_from(skip);
    bool longer = false;
    for (uint32_t i = threadIdx.x; i + kRunCap < n; i += kOneThreads)
      longer |= (slot[i] >> skip) == (slot[i + kRunCap] >> skip);
    every_bit = __syncthreads_or(longer ? 1 : 0) != 0;
  }
  if (every_bit) sort_from(0);
  for (uint32_t i = threadIdx.x; i < n; i += kOneThreads) order[i] = L.vals[i];
  if (threadIdx.x == 0) *full = every_bit ? 1u : 0u;
}

bool one_tile(const Plan &p) {
  // (a shape of four keys a thread is only ever picked by the library)
  return p.nsets == 1 && p.n <= 8 * kOneThreads && p.sort.ipt == 4 &&
         !(p.flags & (TB_SORT_LOOKBACK | TB_SORT_COUNTED));
}

hipError_t launch_sort_one(const Plan &p, const Work &w, const tb_tree &out, hipStream_t s) {
  auto k = p.n <= kOneThreads       ? k_sort_one<1>
           : p.n <= 2 * kOneThreads ? k_sort_one<2>
           : p.n <= 4 * kOneThreads ? k_sort_one<4>
                                    : k_sort_one<8>;
  k<<<1, kOneThreads, 0, s>>>(static_cast<const uint64_t *>(w.keys0), sorted_order(p, w, out),
                              (uint32_t)p.n, p.skip_bits, reorder_finishes(p.n_leaf) ? 0 : 1,
                              w.counters + kFullSortCounter);
  return hipGetLastError();
}

#define TB_SORT_SHAPES(CASE)                                                        \
  CASE(8, 11, 512) CASE(8, 12, 512) CASE(8, 10, 512) CASE(8, 16, 256) CASE(9, 16, 256) \
  CASE(8, 12, 256) CASE(8, 8, 512) CASE(8, 4, 512) CASE(8, 4, 1024)

hipError_t launch_sort_pass(const Plan &p, const Work &w, int pass, const tb_tree &out,
                            hipStream_t s) {
  const SortConfig &c = p.sort;
#define TB_SORT_CASE(B, I, T)                                         \
  if (c.bits == B && c.ipt == I && c.threads == T)                    \
    return launch_pass_t<B, I, T>(p, w, pass, out, s);
  TB_SORT_SHAPES(TB_SORT_CASE)
#undef TB_SORT_CASE
  return hipErrorInvalidValue;
}

hipError_t launch_low_passes(const Plan &p, const Work &w, const tb_tree &out, hipStream_t s) {
  const SortConfig &c = p.sort;
#define TB_SORT_CASE(B, I, T)                                         \
  if (c.bits == B && c.ipt == I && c.threads == T) return launch_low_t<B, I, T>(p, w, out, s);
  TB_SORT_SHAPES(TB_SORT_CASE)
#undef TB_SORT_CASE
  return hipErrorInvalidValue;
}

bool sort_config_supported(const SortConfig &c) {
  static const int table[][3] = {{8, 11, 512}, {8, 12, 512}, {8, 10, 512}, {8, 16, 256},
                                 {9, 16, 256}, {8, 12, 256}, {8, 8, 512}};
  for (const auto &r : table)
    if (r[0] == c.bits && r[1] == c.ipt && r[2] == c.threads) return true;
  return false;
}

}  // namespace tb
