// Top-B selection over the flattened heads of a layer (Alg. 1, "B_l largest entries based on
// s_l"; the per-head survivor counts are the dynamic head budgets of Sec. 4.1).
//
// The paper's cost statement assumes a min-heap, O(H N log B_l); on a GPU the same result comes from
// narrowing an interval of an order-preserving integer image of the score ("key") until it holds the
// threshold key T and little else: a histogram over 1024 intervals of the whole key range (sel_digit0)
// finds the one in which the cumulative count, from the top, reaches the budget; if that interval holds
// few keys (the usual case) every workgroup collects them all and finds T among them in its own LDS,
// otherwise its keys are counted again by their next 10 bits, as often as it takes.  (An end bin of the first
// histogram has its next one counted along with it, see kEndShift.)  Ties at T are
// resolved by ascending flat index with an ordered scan, so the survivor set is unique and the output
// needs no floating-point comparison at all.  Survivors are written in flat order, which is exactly
// "heads concatenated, ascending position inside each head".
//
// The selection is latency-bound (a few MiB of scores): what counts is the number of dependent trips to
// memory and of waits for other workgroups.  It runs as ONE kernel over workgroups of 1024 lanes with KP
// keys per lane in registers.  A problem that fits one workgroup exchanges nothing at all.  Otherwise a
// prepared problem (first histogram built by the score kernels) waits for the other workgroups once, an
// unprepared one twice (its first histogram, then the interval's keys); every workgroup derives T and its
// output offset redundantly, so none waits for a leader.  Inputs too large for all workgroups to be
// resident at once run the same phases as separate kernels.
// Measured (kernel trace, prepared, against three 11-bit digits with a grid-wide wait each and 16 keys per lane):
// 2 K entries 18.9 -> 7.8 us, 33 K 23.3 -> 10.3, 262 K 24.0 -> 12.5, 1 M 26.8 -> 16.7; a step of a cascade
// (several problems, not prepared) 28 -> 18.  Inside the kernel at 262 K, not prepared, n/100: scores in and
// counted 5.1 us (0.5 of it the loads, 3.2 the wait), pick 0.5, split 0.8, exchange 3.0, list 1.0, threshold 1.5,
// write 2.2; a row of keys per lane costs 0.3 us of vector work in all, which is why a lane holds few.
// Calls in a loop, not prepared (three digits -> now, budget n/100 and n/4): 1 M entries, plateaus 31.6 -> 25.8 and
// 32.4 -> 30.2, within 10 % of each other 34.3 -> 29.2 and 35.4 -> 32.3, near 2^-60 32.5 -> 29.9 and 34.0 -> 33.0;
// 4 M as step launches 53 -> 41 .. 44 and 60 -> 46 .. 48; 16 M 160 -> 116 and 176 -> 134.  Behind by 1 to 3 % between
// 1.2 M and 2 M entries, n/4, for scores within 2 % of each other or out of the first histogram's range (1.5 M: 36.3 ->
// 36.9, 37.1 -> 37.6).  Behind for a prepared selection whose threshold lies below 2^-44 or above 2^20, from
// 1 M to 3 M entries: two further histograms (1 M: 27 -> 36; counting the ends in the score kernels as well made
// this 24, and every scores call 0.3 to 1.1 us longer).
#include <type_traits>

#include "common.h"
#include "xblock.h"

namespace lava {

constexpr int kMaxHeads = 64;
constexpr int kLevelBits = 10;
constexpr int kLevelBins = 1 << kLevelBits;
static_assert(kLevelBins == kSelThreads && kSelDigit0Bins == kLevelBins, "one bin per thread");
constexpr unsigned int kSpinLimit = 1u << 18;           // polls of a wait for other workgroups before giving up (default)
constexpr unsigned int kListCap = 16384;                // keys of the threshold's interval a workgroup collects in LDS
constexpr int kFusedMaxBlocks = 512;                    // workgroups of a problem in the one-launch selection

// The first histogram's end bins hold whatever lies beyond its range.  A selection that counts it itself (one that is not
// prepared) counts their keys a second time, by their offset from the bin's lowest key in steps of half an octave: the
// next histogram of either end bin, without another pass and another wait for the other workgroups.  Bins of the low
// end from word 0 on, of the high end from kEndHigh on; the last word is where entries beyond the end go.
constexpr int kEndShift = 32 - kLevelBits;
constexpr int kEndHigh = 768;
constexpr unsigned int kHighLo = kSelKeyBase + ((unsigned int)(kLevelBins - 1) << kSelDigit0Shift);   // lowest key of the last bin
static_assert(((kSelKeyBase + (1u << kSelDigit0Shift) - 2u) >> kEndShift) < kEndHigh &&
              kEndHigh + ((0xffffffffu - kHighLo) >> kEndShift) < kLevelBins - 1, "both ends fit");

// The region's histogram area (3 * kSelBins words, zeroed beforehand): the first histogram, if not prepared the end
// bins' one, the further ones (at most four: 32 bits, or three: 22), then one 64-bit word per workgroup of the one-launch selection.
__device__ __forceinline__ constexpr int next_hist_word(bool primed) { return primed ? kLevelBins : 2 * kLevelBins; }
constexpr int kFlagWord = 5 * kLevelBins;
static_assert(kFlagWord + 2 * kFusedMaxBlocks <= 3 * kSelBins, "histogram area");

struct SelectState {
  unsigned int barrier;      // arrivals at the grid barriers of the fused kernel (monotonic)
  unsigned int error;        // set when a wait gave up (results are then invalid)
  unsigned int outcome;      // kOpen until the fused kernel's workgroups agree on kComplete or kFailed (see there)
  unsigned int reserved[5];
};
constexpr unsigned int kOpen = 0u, kComplete = 1u, kFailed = 2u;
static_assert(sizeof(SelectState) == kSelStateWords * sizeof(unsigned int), "cleared word by word by the score kernels");

SelectWorkspace make_select_workspace(int64_t total) { return select_layout(total); }

struct SelShared {
  unsigned int list[kListCap];              // keys of the threshold's interval, all workgroups', in workgroup order
  unsigned int hist[kLevelBins];
  unsigned int seg_pos[kFusedMaxBlocks + 1];// where workgroup b's keys start in `list`
  int off[kMaxHeads + 1];                   // segment starts
  unsigned int cnt[kMaxHeads];              // survivors per head in this workgroup
  unsigned int wave[kSelWaves];
  unsigned int wave2[kSelWaves];
  unsigned int pick[3];
  unsigned int before[4];                   // handed from wavefront 0 to the workgroup
  unsigned int failed;
};

// The keys that may still hold the threshold: lo .. lo + width.  `need` survivors must come from the
// `count` keys in it, everything above it survives.  2^bits > width.
struct Interval {
  unsigned int lo, width, bits, need, count;
};

__device__ __forceinline__ long long effective_budget(long long budget, const int64_t* budget_dev,
                                                      long long total) {
  long long b = budget;
  if (budget_dev != nullptr) {
    const long long d = (long long)*budget_dev;
    b = d < b ? d : b;
  }
  if (b > total) b = total;
  if (b < 0) b = 0;
  return b;
}

// With explicit segments the number of entries is whatever the last offset says (read on the
// device, so that a caller can chain selections without a host round trip); the host value is then
// an upper bound that sized the grid and the workspace.
__device__ __forceinline__ long long device_total(long long bound, const int64_t* __restrict__ seg_offsets,
                                                  int n_heads) {
  if (seg_offsets == nullptr) return bound;
  long long t = (long long)seg_offsets[n_heads];
  t = t < 0 ? 0 : t;
  return t < bound ? t : bound;
}

// First entry of head h (h == n_heads: the end), in the range of an int whatever the caller's table holds.
__device__ __forceinline__ int segment_start(const int64_t* __restrict__ seg_offsets, int h, int n_heads, int total) {
  if (seg_offsets == nullptr) return h == n_heads ? total : total / n_heads * h;
  const long long p = (long long)seg_offsets[h];
  return p < 0 ? 0 : (p > 0x7fffffffll ? 0x7fffffff : (int)p);
}

// A workgroup's keys: wavefront w holds the 64 * KP consecutive entries from wave_base on as KP rows of
// 64 (row j, lane l: entry wave_base + 64 j + l), so that loads are coalesced whatever the alignment of
// the scores and the flat order inside a wavefront is row by row, lane by lane: positions are bit counts
// of ballots, nothing goes through LDS.  Entries beyond the end get key 0, which no entry has: the one score
// whose image it is, the NaN with all bits set, gets 1, so that it is ranked like any other (NaN is no valid score,
// but a slot counted and not written would be an index from nowhere for the gather behind the selection).  One loop maps
// the keys of complete and of partly filled wavefronts: a loop in either branch cost 4 us of a 16-sequence batch.
template <int KP>
__device__ __forceinline__ void load_keys(const float* __restrict__ scores, int wave_base, int total,
                                          unsigned int (&key)[KP]) {
  const int lane = (int)(threadIdx.x & 63);
  const bool complete = span_complete(wave_base, 64 * KP, total);
  if (complete) {                                   // uniform; all loads in flight before the first use
    const float* __restrict__ src = scores + wave_base + lane;
#pragma unroll
    for (int j = 0; j < KP; ++j) key[j] = __float_as_uint(src[64 * j]);
  } else {
#pragma unroll
    for (int j = 0; j < KP; ++j) {
      const int p = wave_base + lane + 64 * j;
      key[j] = p < total ? __float_as_uint(scores[p]) : 0u;
    }
  }
#pragma unroll
  for (int j = 0; j < KP; ++j) {
    const unsigned int k = score_key(__uint_as_float(key[j]));
    key[j] = k > 1u ? k : 1u;
  }
  if (!complete) {
#pragma unroll
    for (int j = 0; j < KP; ++j) key[j] = wave_base + lane + 64 * j < total ? key[j] : 0u;
  }
}
static_assert(kMaxHeads <= 64, "one lane per head");

// Entries of workgroup bx's chunk that lie beyond the end.
template <int KP>
__device__ __forceinline__ unsigned int missing(int bx, int total) {
  const long long end = (long long)(bx + 1) * (kSelThreads * KP), over = end - total;
  return over <= 0 ? 0u : (over < kSelThreads * KP ? (unsigned int)over : (unsigned int)(kSelThreads * KP));
}

// A uniform value the compiler cannot connect with its earlier uses: row masks that are formed twice are
// compared twice instead of being kept in (spilled) scalar registers from one loop to the other.
__device__ __forceinline__ unsigned int opaque(unsigned int x) {
  x = __builtin_amdgcn_readfirstlane(x);
  asm volatile("" : "+s"(x));
  return x;
}

__device__ __forceinline__ unsigned int level_shift(const Interval& v) {
  return v.bits > (unsigned int)kLevelBits ? v.bits - kLevelBits : 0u;
}
// LDS add whose result nobody needs, as an instruction: the compiler would turn an atomic add into a
// reduction over the lanes first, which costs more than the add.
__device__ __forceinline__ unsigned int lds_offset(const void* p) {
  return (unsigned int)(unsigned long long)(__attribute__((address_space(3))) const char*)p;
}
__device__ __forceinline__ void lds_add(unsigned int at, unsigned int x) {
  asm volatile("ds_add_u32 %0, %1" : : "v"(at), "v"(x) : "memory");
}

// every LDS operation of this wavefront is complete
__device__ __forceinline__ void lds_done() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

// Keeps the compiler from forming the masks of many rows ahead of their use (they do not fit the scalar registers).
__device__ __forceinline__ void row_done() { __builtin_amdgcn_sched_barrier(0); }

// One count for every lane's bin (byte address in LDS).  A row in one bin (a large plateau: zeros, the window
// entries) is one add.
__device__ __forceinline__ void count_row(unsigned int at) {
  const unsigned int at0 = __builtin_amdgcn_readfirstlane(at);
  if (__all(at == at0)) {
    if ((threadIdx.x & 63) == 0) lds_add(at0, 64u);
  } else {
    lds_add(at, 1u);
  }
  row_done();
}

// ... for the lanes inside the interval that is counted.  The others stay out of it altogether: a bin for them
// that nobody reads takes up to 64 adds to one address, one after the other (1 M entries, budget n/4, scores within
// 10 % of each other: 9.3 us for this histogram, 1.9 without such a bin; 41.6 -> 34.2 for the call, 4 M 83 -> 63.7).
__device__ __forceinline__ void count_row(bool in, unsigned int at) {
  const unsigned long long lanes = __ballot(in);
  if (lanes != 0ull) {                                        // uniform
    const int leader = __builtin_ctzll(lanes);
    const unsigned int at0 = (unsigned int)__builtin_amdgcn_readlane((int)at, leader);
    if (__ballot(in && at == at0) == lanes) {
      if ((int)(threadIdx.x & 63) == leader) lds_add(at0, (unsigned int)__popcll(lanes));
    } else if (in) {
      lds_add(at, 1u);
    }
  }
  row_done();
}

// First histogram (bins sel_digit0) over this wavefront's keys, in `hist`, and the end bins' one in `ends` (LDS; zeroed
// and published by a barrier before).  Entries beyond the end have key 0, i.e. count in bin 0: the caller takes them out again.
// The keys of an end bin are counted there per row and not per lane, which would be one address for many.
template <int KP>
__device__ __forceinline__ void count_first(const unsigned int (&key)[KP], unsigned int* hist, unsigned int* ends) {
  constexpr unsigned int kFirst = kSelKeyBase >> kSelDigit0Shift, kLast = kFirst + kSelDigit0Bins - 1u;
  static_assert((kFirst << kSelDigit0Shift) == kSelKeyBase, "bins are aligned in the key");
  const unsigned int base = lds_offset(hist) - 4u * kFirst, ends_at = lds_offset(ends);
#pragma unroll
  for (int j = 0; j < KP; ++j) {
    unsigned int d = key[j] >> kSelDigit0Shift;
    d = d < kFirst ? kFirst : d;
    d = d > kLast ? kLast : d;
    unsigned int at = base + 4u * d;
    const bool end = d - (kFirst + 1u) > kLast - kFirst - 2u;
    const unsigned long long in_ends = __ballot(end);
    if (in_ends != 0ull) {                                    // uniform
      const unsigned long long low = __ballot(d == kFirst);
      if ((threadIdx.x & 63) == 0) {
        lds_add(base + 4u * kFirst, (unsigned int)__popcll(low));
        lds_add(base + 4u * kLast, (unsigned int)__popcll(in_ends & ~low));
      }
      const unsigned int of_end = d == kFirst ? (key[j] - 1u) >> kEndShift : kEndHigh + ((key[j] - kHighLo) >> kEndShift);
      if (end) at = ends_at + 4u * of_end;
    }
    count_row(at);
  }
}

// Histogram of the keys inside interval v by their next bits.
template <int KP>
__device__ __forceinline__ void count_level(const unsigned int (&key)[KP], const Interval& v, unsigned int* hist) {
  const unsigned int shift = level_shift(v), base = lds_offset(hist);
#pragma unroll
  for (int j = 0; j < KP; ++j) {
    const unsigned int rel = key[j] - v.lo;
    count_row(rel <= v.width, base + 4u * (rel >> shift));
  }
}

// Sums across lanes without LDS: data-parallel-primitive moves (a shift inside rows of 16 lanes, then the last
// lane of one row to the next ones), a few cycles each where a shuffle is a trip through the LDS unit.
template <int CTRL, int ROWS>
__device__ __forceinline__ unsigned int dpp_add(unsigned int x) {
  return x + (unsigned int)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, ROWS, 0xf, false);
}
__device__ __forceinline__ unsigned int row_scan(unsigned int x) {        // inclusive, inside each row of 16 lanes
  x = dpp_add<0x111, 0xf>(x);
  x = dpp_add<0x112, 0xf>(x);
  x = dpp_add<0x114, 0xf>(x);
  return dpp_add<0x118, 0xf>(x);
}
__device__ __forceinline__ unsigned int wave_scan(unsigned int x) {       // inclusive, over the wavefront
  x = row_scan(x);
  x = dpp_add<0x142, 0xa>(x);
  return dpp_add<0x143, 0xc>(x);
}
__device__ __forceinline__ unsigned int wave_sum(unsigned int x) {
  return (unsigned int)__builtin_amdgcn_readlane((int)wave_scan(x), 63);
}
// One word per wavefront in LDS: their sum, and that of the wavefronts before `wave`.
struct WaveSums {
  unsigned int total, before;
};
__device__ __forceinline__ WaveSums wave_sums(const unsigned int* w, int wave) {
  static_assert(kSelWaves == 16, "one row of lanes");
  const unsigned int mine = w[threadIdx.x & 15], incl = row_scan(mine);
  WaveSums r;
  r.total = (unsigned int)__builtin_amdgcn_readlane((int)incl, 15);
  r.before = (unsigned int)__builtin_amdgcn_readlane((int)(incl - mine), wave);
  return r;
}
// Index of this wavefront, as a scalar.
__device__ __forceinline__ int sel_wave() { return __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)); }

// The bin, counted from the top, in which the cumulative count reaches `need` (> 0); `mine` is the count
// of bin kLevelBins - 1 - threadIdx.x.  Returns (bin, survivors needed from it, its count) in `out`.
__device__ __forceinline__ void pick_bin(unsigned int mine, unsigned int need, SelShared& sh, unsigned int (&out)[3]) {
  const unsigned int incl = wave_scan(mine);
  const int wave = sel_wave();
  if ((threadIdx.x & 63) == 63) sh.wave[wave] = incl;
  if (threadIdx.x == 0) { sh.pick[0] = 0u; sh.pick[1] = need; sh.pick[2] = 0u; }   // taken only if the counts are short of `need` (a wait gave up)
  __syncthreads();
  const unsigned int above = wave_sums(sh.wave, wave).before + incl - mine;
  if (above < need && need <= above + mine) {
    sh.pick[0] = (unsigned int)(kLevelBins - 1) - threadIdx.x;
    sh.pick[1] = need - above;
    sh.pick[2] = mine;
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 3; ++i) out[i] = __builtin_amdgcn_readfirstlane(sh.pick[i]);
}

// Interval of the first histogram's bin.
__device__ __forceinline__ Interval first_interval(const unsigned int (&pk)[3]) {
  Interval v;
  v.lo = pk[0] == 0u ? 1u : kSelKeyBase + (pk[0] << kSelDigit0Shift);      // the end bins take whatever lies beyond
  const unsigned int hi = pk[0] == (unsigned int)(kLevelBins - 1) ? 0xffffffffu
                                                                 : kSelKeyBase + ((pk[0] + 1u) << kSelDigit0Shift) - 1u;
  v.width = hi - v.lo;
  v.bits = (pk[0] == 0u || pk[0] == (unsigned int)(kLevelBins - 1)) ? 32u : (unsigned int)kSelDigit0Shift;
  v.need = pk[1];
  v.count = pk[2];
  return v;
}
__device__ __forceinline__ void narrow(Interval& v, const unsigned int (&pk)[3]) {
  const unsigned int sh = level_shift(v), skip = pk[0] << sh, most = (1u << sh) - 1u;
  v.lo += skip;
  v.width = v.width - skip < most ? v.width - skip : most;
  v.bits = sh;
  v.need = pk[1];
  v.count = pk[2];
}

// The interval of an end bin (`low`: the first one) narrowed by the histogram of the ends in `ends`; READ: how to read
// a word of it.  Contains workgroup barriers.
template <class READ>
__device__ __forceinline__ void narrow_end(Interval& v, bool low, SelShared& sh, READ&& read) {
  const int bin = kLevelBins - 1 - (int)threadIdx.x, word = low ? bin : kEndHigh + bin;
  const unsigned int mine = word < (low ? kEndHigh : kLevelBins - 1) ? read(word) : 0u;
  __syncthreads();                                   // sh.pick has been read
  unsigned int pk[3];
  pick_bin(mine, v.need, sh, pk);
  narrow(v, pk);
}

// What a survivor is: key > T, or key == T and among the first `ties` such keys in flat order.
struct Threshold {
  unsigned int T, ties;
};
// ... once the interval is one key wide, or all of its keys survive
__device__ __forceinline__ bool decided(const Interval& v) { return v.bits == 0u || v.count == v.need; }
__device__ __forceinline__ Threshold threshold_of(const Interval& v) {
  Threshold t;
  const bool all = v.count == v.need;
  t.T = all ? v.lo - 1u : v.lo;                    // lo >= 1
  t.ties = all ? 0u : v.need;
  return t;
}

// Ordered write of this workgroup's survivors, which lie in `rows` of its wavefronts (bit j: row j; gt_wg keys
// above T and eq_wg equal to T lie in the workgroups before it);
// survivors per head go to head_counts, head offsets are written by the wavefront that holds the first
// entry of the head.  Contains workgroup barriers.
template <int KP>
__device__ __forceinline__ void write_survivors(const unsigned int (&key)[KP], unsigned int rows, const float* __restrict__ scores,
                                                int wave_base, int total, int n_heads, Threshold t,
                                                unsigned int gt_wg, unsigned int eq_wg, int kept_total, long long capacity,
                                                bool alone, bool first_wg, SelShared& sh,
                                                int32_t* __restrict__ head_counts, int64_t* __restrict__ head_offsets,
                                                int32_t* __restrict__ kept_idx, float* __restrict__ kept_scores) {
  const int lane = threadIdx.x & 63, wave = sel_wave();
  // lane j: which keys of row j lie above T / are equal to it
  unsigned long long row_gt = 0ull, row_eq = 0ull;
#pragma unroll
  for (int j = 0; j < KP; ++j) {
    if (!((rows >> j) & 1u)) continue;                        // uniform
    const unsigned long long gt = __ballot(key[j] > t.T), eq = t.ties ? __ballot(key[j] == t.T) : 0ull;
    if (lane == j) { row_gt = gt; row_eq = eq; }
    row_done();
  }
  const unsigned int mine = ((unsigned int)__popcll(row_gt) << 16) | (unsigned int)__popcll(row_eq);
  const unsigned int incl = wave_scan(mine);
  if (lane == 63) sh.wave2[wave] = incl;
  if (threadIdx.x < kMaxHeads) sh.cnt[threadIdx.x] = 0u;
  __syncthreads();
  static_assert(64 * KP * (kSelWaves - 1) < (1 << 16) && KP <= 32, "packed counts, one lane per row");
  const unsigned int base = wave_sums(sh.wave2, wave).before, excl = incl - mine;
  const unsigned int gt_wave = gt_wg + (base >> 16), eq_wave = eq_wg + (base & 0xffffu);
  const unsigned int row_gt0 = gt_wave + (excl >> 16), row_eq0 = eq_wave + (excl & 0xffffu);   // lane j: keys before row j

  // survivors before entry p of this wavefront (p uniform)
  auto survivors_before = [&](int p) -> unsigned int {
    const int r = (p - wave_base) >> 6, l = (p - wave_base) & 63;
    const unsigned long long below = (1ull << l) - 1ull;
    const unsigned int gt = row_gt0 + (unsigned int)__popcll(row_gt & below);
    unsigned int eq = row_eq0 + (unsigned int)__popcll(row_eq & below);
    if (eq > t.ties) eq = t.ties;
    return (unsigned int)__builtin_amdgcn_readlane((int)(gt + eq), r);
  };
  const unsigned int all = (unsigned int)__builtin_amdgcn_readlane((int)incl, 63);
  const unsigned int eq0 = eq_wave < t.ties ? eq_wave : t.ties;
  const unsigned int eq1 = eq_wave + (all & 0xffffu) < t.ties ? eq_wave + (all & 0xffffu) : t.ties;
  const unsigned int s_begin = gt_wave + eq0, s_end = gt_wave + (all >> 16) + eq1;

  // heads that start inside this wavefront's entries
  const int start = lane < n_heads ? sh.off[lane] : 0x7fffffff;
  const unsigned long long started = __ballot(lane < n_heads && start <= wave_base);
  int g = started ? 63 - __builtin_clzll(started) : 0;        // head of the wavefront's first entry
  const int g_first = g;
  const bool here = lane > 0 && lane < n_heads && in_span(start, wave_base, 64 * KP);
  unsigned long long starts = __ballot(here && start < total);
  const bool several = __ballot(here && start > wave_base) != 0ull;
  unsigned int s_prev = s_begin;
  while (starts) {
    const int h = __builtin_ctzll(starts);
    starts &= starts - 1ull;
    const int p = __builtin_amdgcn_readlane(start, h);
    const unsigned int s = survivors_before(p);
    if (lane == 0) {
      head_offsets[h] = (int64_t)s;
      if (p > wave_base && s != s_prev) atomicAdd(&sh.cnt[g], s - s_prev);
    }
    if (p > wave_base) { s_prev = s; g = h; }
  }
  if (lane == 0 && s_end != s_prev) atomicAdd(&sh.cnt[g], s_end - s_prev);
  // the two ends, and heads that start at or beyond the end (empty trailing heads)
  if (first_wg && threadIdx.x < 64) {
    if (lane == 0) head_offsets[n_heads] = (int64_t)kept_total;
    if (lane == 0) head_offsets[0] = 0;
    if (lane > 0 && lane < n_heads && start >= total) head_offsets[lane] = (int64_t)kept_total;
  }

  const int head_start = __builtin_amdgcn_readlane(start, g_first);
  rows = (unsigned int)__ballot((row_gt | row_eq) != 0ull);
  const unsigned int T = opaque(t.T);
#pragma unroll
  for (int j = 0; j < KP; ++j) {
    if (!((rows >> j) & 1u)) continue;                        // uniform
    const bool is_gt = key[j] > T, is_eq = t.ties != 0u && key[j] == T;
    const unsigned long long gt = __ballot(is_gt), eq = __ballot(is_eq);
    const unsigned int gt_rank = (unsigned int)__builtin_amdgcn_readlane((int)row_gt0, j) +
                                 __builtin_amdgcn_mbcnt_hi((unsigned int)(gt >> 32), __builtin_amdgcn_mbcnt_lo((unsigned int)gt, 0u));
    const unsigned int eq_rank = (unsigned int)__builtin_amdgcn_readlane((int)row_eq0, j) +
                                 __builtin_amdgcn_mbcnt_hi((unsigned int)(eq >> 32), __builtin_amdgcn_mbcnt_lo((unsigned int)eq, 0u));
    if (is_gt || (is_eq && eq_rank < t.ties)) {
      const long long slot = (long long)gt_rank + (eq_rank < t.ties ? eq_rank : t.ties);
      if (slot < capacity) {
        const int p = wave_base + 64 * j + lane;
        int from = head_start;
        if (several) {                                        // the last head that starts at or before p
          int h = g_first;
          while (h + 1 < n_heads && sh.off[h + 1] <= p) ++h;
          from = sh.off[h];
        }
        kept_idx[slot] = p - from;
        if (kept_scores) {
          // the score behind a key; both zeros share one and a NaN's bits are not all kept, so those are read again
          constexpr unsigned int kLowest = 0x007fffffu, kHighest = 0xff800000u;      // keys of -inf and +inf
          const unsigned int k = key[j];
          float f = __uint_as_float((k & 0x80000000u) ? (k ^ 0x80000000u) : ~k);
          if (k == 0x80000000u || k - kLowest > kHighest - kLowest) f = scores[p];
          kept_scores[slot] = f;
        }
      }
    }
  }
  __syncthreads();
  if (threadIdx.x < n_heads) {
    const unsigned int c = sh.cnt[threadIdx.x];
    if (alone) head_counts[threadIdx.x] = (int32_t)c;
    else if (c) __hip_atomic_fetch_add(reinterpret_cast<unsigned int*>(&head_counts[threadIdx.x]), c,
                                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

// Grid-wide barrier of the fused kernel: all of its workgroups are resident (the host checks the
// grid against the device's capacity), arrivals are counted monotonically, and the wait is
// bounded: if it ever gives up, the outcome is failure and the kernel still runs to completion.
__device__ __forceinline__ void grid_sync(SelectState* __restrict__ st, unsigned int round, unsigned int n_blocks,
                                          unsigned int spin_limit) {
  drain_vmem();
  __syncthreads();
  if (threadIdx.x == 0) {
    __hip_atomic_fetch_add(&st->barrier, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const unsigned int target = round * n_blocks;
    unsigned int spins = 0u;
    while (ld_dev(&st->barrier) < target) {
      __builtin_amdgcn_s_sleep(2);
      if (++spins > spin_limit) {
        st_dev(&st->outcome, kFailed);       // still open: this workgroup's keys are not published yet
        break;
      }
    }
  }
  __syncthreads();
}

// One launch serves up to kMaxSelProblems independent selections: the table travels in the kernel
// arguments, and the workgroups of all problems are numbered through (first_block), so every
// workgroup of the grid has work.  Every problem has its own histograms, barrier counter and
// exchange words in its own region of the workspace, so problems never wait for each other.
struct SelectBatch {
  int n_heads;
  int n_problems;
  int first_block[kMaxSelProblems + 1];   // workgroups of problem p: first_block[p] .. first_block[p + 1] - 1
  char* ws;                      // region of problem p at ws + p * ws_stride
  size_t ws_stride, off_hist, off_state, off_blk;
  unsigned int spin_limit;       // polls of a wait for other workgroups before it gives up
  unsigned int seg_words;        // one-launch selection: words of a workgroup's segment
  unsigned int primed_mask;      // bit p: problem p's region was prepared by the score kernels (first histogram
                                 // complete, the rest cleared)
  lava_select_problem p[kMaxSelProblems];
};

// Problem of this workgroup (uniform over the workgroup).
__device__ __forceinline__ int problem_of_block(const SelectBatch& a) {
  if (a.n_problems == 1) return 0;
  const int lane = threadIdx.x & 63;
  const unsigned long long at = __ballot(lane < a.n_problems && a.first_block[lane < a.n_problems ? lane : 0] <= (int)blockIdx.x);
  return 63 - __builtin_clzll(at);                // first_block[0] = 0
}
static_assert(kMaxSelProblems <= 64, "one lane per problem");

__global__ void __launch_bounds__(kSelThreads) sel_init_kernel(const SelectBatch a) {
  const lava_select_problem pr = a.p[blockIdx.x];
  char* region = a.ws + blockIdx.x * a.ws_stride;
  unsigned int* hist = reinterpret_cast<unsigned int*>(region + a.off_hist);
  SelectState* st = reinterpret_cast<SelectState*>(region + a.off_state);
  if (threadIdx.x < a.n_heads) pr.head_counts[threadIdx.x] = 0;
  if ((a.primed_mask >> blockIdx.x) & 1u) return;           // histograms and state are as the score kernels left them
  for (int i = threadIdx.x; i < 3 * kSelBins; i += kSelThreads) hist[i] = 0u;
  if (threadIdx.x == 0) {
    st->barrier = 0u;
    st->error = 0u;
    st->outcome = kOpen;
  }
}

// The keys of the threshold's interval that lie in this workgroup: how many keys lie above the interval
// and in it (out: the workgroup's sums; `base`: those of the wavefronts before this one), and row by row
// which ones.  Contains a workgroup barrier.
template <int KP>
__device__ __forceinline__ void split_keys(const unsigned int (&key)[KP], const Interval& v, SelShared& sh, unsigned int& above,
                                           unsigned int& inside, unsigned int& inside_base,
                                           unsigned int& rows_above, unsigned int& rows_inside) {
  const int wave = sel_wave();
  const unsigned int hi = v.lo + v.width;
  unsigned int n_above = 0u, n_inside = 0u;                   // scalar: the wavefront's
  rows_above = rows_inside = 0u;
#pragma unroll
  for (int j = 0; j < KP; ++j) {
    const unsigned long long up = __ballot(key[j] > hi), in = __ballot(key[j] - v.lo <= v.width);
    n_above += (unsigned int)__popcll(up);
    n_inside += (unsigned int)__popcll(in);
    rows_above |= up ? 1u << j : 0u;
    rows_inside |= in ? 1u << j : 0u;
    row_done();
  }
  if ((threadIdx.x & 63) == 0) sh.wave2[wave] = (n_above << 16) | n_inside;    // at most 32768 in all
  __syncthreads();
  const WaveSums sums = wave_sums(sh.wave2, wave);
  above = sums.total >> 16;
  inside = sums.total & 0xffffu;
  inside_base = sums.before & 0xffffu;
}

// put(position, key) for this wavefront's keys of the interval, in flat order from position `at` on.
template <int KP, class F>
__device__ __forceinline__ void collect_keys(const unsigned int (&key)[KP], const Interval& v, unsigned int at,
                                             unsigned int rows_inside, F&& put) {
  const unsigned int lo = opaque(v.lo), width = v.width;
#pragma unroll
  for (int j = 0; j < KP; ++j) {
    if (!((rows_inside >> j) & 1u)) continue;                 // uniform
    const bool in = key[j] - lo <= width;
    const unsigned long long b = __ballot(in);
    if (in) put(at + __builtin_amdgcn_mbcnt_hi((unsigned int)(b >> 32), __builtin_amdgcn_mbcnt_lo((unsigned int)b, 0u)), key[j]);
    at += (unsigned int)__popcll(b);
  }
}

// The keys of all workgroups' segments into sh.list.  A wavefront takes a run of the list: its lanes look up the segment
// of their first entry and walk on from there, a word of LDS for every segment they pass, with kListAhead loads in
// flight.  (A search for every entry in front of its load took 8.2 us
// for 15 K keys in 86 segments, this takes 2.7: 1 M entries, budget n/4, 35.2 -> 32.7 for the call.)
constexpr unsigned int kListAhead = 4u;
__device__ __forceinline__ void fetch_list(const unsigned int* seg, unsigned int seg_words, unsigned int nb, unsigned int n_list,
                                           SelShared& sh) {
  const unsigned int run = (n_list + kSelThreads - 1u) / kSelThreads * 64u;      // 64 entries a step
  const unsigned int begin = (unsigned int)sel_wave() * run, end = begin + run < n_list ? begin + run : n_list;
  unsigned int i = begin + (threadIdx.x & 63);
  if (i >= end) return;
  unsigned int lo = 0u, hi = nb;                                // the segment that holds entry i
  while (hi - lo > 1u) {
    const unsigned int mid = (lo + hi) >> 1;
    if (sh.seg_pos[mid] <= i) lo = mid; else hi = mid;
  }
  unsigned int from = sh.seg_pos[lo], to = sh.seg_pos[lo + 1u];
  for (; i < end; i += 64u * kListAhead) {
    unsigned int k[kListAhead];
#pragma unroll
    for (unsigned int u = 0; u < kListAhead; ++u) {
      const unsigned int at = i + 64u * u;
      if (at < end) {
        while (at >= to) { ++lo; from = to; to = sh.seg_pos[lo + 1u]; }       // at < n_list <= seg_pos[nb]
        k[u] = ld_dev(&seg[lo * seg_words + (at - from)]);
      }
    }
#pragma unroll
    for (unsigned int u = 0; u < kListAhead; ++u)
      if (i + 64u * u < end) sh.list[i + 64u * u] = k[u];
  }
}

// What becomes of a selection whose waits are bounded: either every workgroup writes its survivors or every one writes
// the mark no consumer can mistake for a selection (no survivors anywhere, counts -1).  The first proposal stands: a
// workgroup that has seen the words of all others in the last exchange proposes completion, one whose wait is over its
// limit failure; one that is outvoted by completion finds the words in place.  A wait before that fails while the outcome is
// open, and its failure is visible before the word that the others wait for.  The answer is not needed before the survivors
// are written, so it travels beside the rest of the selection.  (Marks written over the results by the workgroup that
// finishes last, found by a ticket, were two trips to memory and two barriers at the end of every selection:
// 33 K entries 11.1 -> 10.5 us, a cascade step 18.4 -> 17.6.)  For wavefront 0; the outcome before the proposal, in lane 0.
__device__ __forceinline__ unsigned int propose(SelectState* st, unsigned int outcome) {
  unsigned int was = kOpen;
  if ((threadIdx.x & 63) == 0) was = atomicCAS(&st->outcome, kOpen, outcome);
  return was;
}

// The whole selection in one launch.
template <int KP>
__global__ void __launch_bounds__(kSelThreads, 8) sel_fused_kernel(const SelectBatch a) {
  const int prob = problem_of_block(a);
  const lava_select_problem pr = a.p[prob];
  const int bx = (int)blockIdx.x - a.first_block[prob];
  const unsigned int nb = (unsigned int)(a.first_block[prob + 1] - a.first_block[prob]);
  const bool alone = nb == 1u;
  const unsigned int seg_words = a.seg_words;
  char* region = a.ws + prob * a.ws_stride;
  unsigned int* hist = reinterpret_cast<unsigned int*>(region + a.off_hist);
  unsigned long long* flag = reinterpret_cast<unsigned long long*>(hist + kFlagWord);
  SelectState* st = reinterpret_cast<SelectState*>(region + a.off_state);
  unsigned int* seg = reinterpret_cast<unsigned int*>(region + a.off_blk);
  const bool primed = ((a.primed_mask >> prob) & 1u) && !alone;
  __shared__ SelShared sh;

  const int lane = threadIdx.x & 63, wave = sel_wave();
  // a prepared first histogram travels together with the scores
  unsigned int bin_count = 0u;
  if (primed) bin_count = ld_dev(&hist[kLevelBins - 1 - threadIdx.x]);
  const int64_t* __restrict__ seg_offsets = pr.seg_offsets;
  const int n_heads = a.n_heads;
  const long long in_off = pr.in_offset_dev ? (long long)*pr.in_offset_dev : 0;
  const float* __restrict__ scores = pr.scores + in_off;
  const int total = (int)device_total(pr.total_entries, seg_offsets, n_heads);
  const int kept_total = (int)effective_budget(pr.budget, pr.budget_dev, total);
  const int wave_base = __builtin_amdgcn_readfirstlane((bx * kSelWaves + wave) * (64 * KP));
  unsigned int key[KP];
  load_keys<KP>(scores, wave_base, total, key);
  if (threadIdx.x <= n_heads)                        // published by the barriers below
    sh.off[threadIdx.x] = segment_start(seg_offsets, (int)threadIdx.x, n_heads, total);
  if (alone && threadIdx.x == 0) st->error = 0u;     // nothing cleared the region, and nothing here can fail
  // Survivor counts of a prepared problem are cleared here, before this workgroup's exchange word is
  // published: nobody adds to them before having seen all of those (device-scope, as the additions are).
  if (primed && bx == 0 && threadIdx.x < (unsigned)n_heads)
    st_dev(reinterpret_cast<unsigned int*>(&pr.head_counts[threadIdx.x]), 0u);

  bool failed = false;                               // wavefront 0: a wait gave up, here or elsewhere
  unsigned int outcome = kOpen;                      // lane 0 of it: the outcome before this workgroup's proposal
  Threshold t = {0xffffffffu, 0u};                   // nothing survives
  unsigned int rows = 0u;                            // rows of this wavefront that may hold survivors
  unsigned int gt_before = 0u, eq_before = 0u;
  if (kept_total > 0) {                              // uniform over the problem's workgroups, like everything below
    // ---- the first histogram, unless the region was prepared, and the interval that holds the threshold
    unsigned int round = 0u;
    unsigned int pk[3];
    if (!primed) {
      sh.hist[threadIdx.x] = sh.list[threadIdx.x] = 0u;        // sh.list: the end bins' histogram, until keys are collected there
      __syncthreads();
      count_first<KP>(key, sh.hist, sh.list);
      lds_done();
      __syncthreads();
      bin_count = sh.hist[kLevelBins - 1 - threadIdx.x];
      if (threadIdx.x == kLevelBins - 1) bin_count -= missing<KP>(bx, total);
      if (!alone) {
        unsigned int* gh = &hist[(kLevelBins - 1) - threadIdx.x];
        if (bin_count) __hip_atomic_fetch_add(gh, bin_count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const unsigned int of_end = sh.list[threadIdx.x];
        if (of_end) __hip_atomic_fetch_add(&hist[kLevelBins + threadIdx.x], of_end, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        grid_sync(st, ++round, nb, a.spin_limit);
        bin_count = ld_dev(gh);
      }
    }
    pick_bin(bin_count, (unsigned int)kept_total, sh, pk);
    Interval v = first_interval(pk);
    if (!primed && v.bits == 32u && !decided(v))
      narrow_end(v, pk[0] == 0u, sh, [&](int w) { return alone ? sh.list[w] : ld_dev(&hist[kLevelBins + w]); });
    int word = next_hist_word(primed);               // of the next histogram in the region
    bool crowded = false;                            // one workgroup holds more of the interval's keys than its segment takes
    unsigned int epoch = 0u;
    for (;;) {
      // ---- too many keys to collect: count them by their next bits
      while (!decided(v) && (v.count > kListCap || crowded)) {
        __syncthreads();
        sh.hist[threadIdx.x] = 0u;
        __syncthreads();
        count_level<KP>(key, v, sh.hist);
        lds_done();
        __syncthreads();
        bin_count = sh.hist[kLevelBins - 1 - threadIdx.x];
        if (!alone) {
          unsigned int* gh = &hist[word + (kLevelBins - 1) - threadIdx.x];
          if (bin_count) __hip_atomic_fetch_add(gh, bin_count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          grid_sync(st, ++round, nb, a.spin_limit);
          bin_count = ld_dev(gh);
        }
        pick_bin(bin_count, v.need, sh, pk);
        narrow(v, pk);
        word += kLevelBins;
        crowded = false;
      }
      // ---- collect them
      unsigned int above, inside, inside_base;
      unsigned int rows_above, rows_inside;
      split_keys<KP>(key, v, sh, above, inside, inside_base, rows_above, rows_inside);
      rows = rows_above | rows_inside;
      const bool want_keys = !decided(v);
      unsigned int n_list = inside, list_before = 0u;
      if (alone) {
        if (want_keys) collect_keys<KP>(key, v, inside_base, rows_inside, [&](unsigned int at, unsigned int k) { sh.list[at] = k; });   // inside == v.count <= kListCap
      } else {
        // this workgroup's keys to its segment, then its counts; the counts are the signal that the keys are there
        if (want_keys && inside <= seg_words)
          collect_keys<KP>(key, v, inside_base, rows_inside,
                           [&](unsigned int at, unsigned int k) { st_dev(&seg[(unsigned int)bx * seg_words + at], k); });
        drain_vmem();
        __syncthreads();
        ++epoch;
        if (wave == 0) {
          if (lane == 0)
            st_dev(&flag[bx], ((unsigned long long)epoch << 48) | ((unsigned long long)above << 24) | inside);
          unsigned int gt = 0u, before = 0u, pos = 0u, over = 0u, spins = 0u;
          bool patient = false;                        // the words are all there already: somebody has seen them
          for (unsigned int b0 = 0; b0 < nb; b0 += 64u) {
            const unsigned int b = b0 + (unsigned int)lane;
            unsigned long long x = 0ull;
            for (;;) {
              if (b < nb) x = ld_dev(&flag[b]);
              if (__all(b >= nb || (unsigned int)(x >> 48) >= epoch)) break;
              if (failed) break;
              if (!patient && ++spins > a.spin_limit) {
                patient = __builtin_amdgcn_readfirstlane(propose(st, kFailed)) == kComplete;
                failed = !patient;
                if (failed) break;
              }
              __builtin_amdgcn_s_sleep(1);
            }
            if (b >= nb || (unsigned int)(x >> 48) < epoch) x = 0ull;
            const unsigned int ab = (unsigned int)(x >> 24) & 0xffffffu, in = (unsigned int)x & 0xffffffu;
            const unsigned int incl = wave_scan(in);
            if (b < nb) sh.seg_pos[b] = pos + incl - in;
            pos += (unsigned int)__builtin_amdgcn_readlane((int)incl, 63);
            if (b < (unsigned int)bx) { gt += ab; before += in; }
            over |= in > seg_words ? 1u : 0u;
          }
          gt = wave_sum(gt);
          before = wave_sum(before);
          over = __any(over != 0u) ? 1u : 0u;
          // the last exchange: from here on nobody has to wait
          if (!failed && !(want_keys && over != 0u)) outcome = propose(st, kComplete);
          if (lane == 0) {
            sh.seg_pos[nb] = pos;
            sh.before[0] = gt;
            sh.before[1] = before;
            sh.before[2] = over;
            sh.before[3] = pos;
          }
        }
        __syncthreads();
        gt_before = __builtin_amdgcn_readfirstlane(sh.before[0]);
        list_before = __builtin_amdgcn_readfirstlane(sh.before[1]);
        n_list = __builtin_amdgcn_readfirstlane(sh.before[3]);
        crowded = want_keys && __builtin_amdgcn_readfirstlane(sh.before[2]) != 0u;
        if (want_keys && !crowded) {
          if (n_list > kListCap) n_list = kListCap;                       // (only after a wait gave up)
          fetch_list(seg, seg_words, nb, n_list, sh);
        }
      }
      if (!want_keys) {
        t = threshold_of(v);
        if (t.ties) eq_before = list_before;         // all equal to T
        else gt_before += list_before;               // all survive
        break;
      }
      if (crowded) continue;
      // ---- the threshold among the collected keys
      sh.hist[threadIdx.x] = 0u;
      while (!decided(v)) {
        __syncthreads();                             // the histogram is clear; the list is complete
        const unsigned int shift = level_shift(v), base = lds_offset(sh.hist);
        // A run of consecutive entries per thread: equal scores (plateaus of the pooling) then meet in one lane and not in
        // one instruction (1 M entries, budget n/4: 31.2 -> 30.6 us); an odd number, so that lanes read from different banks.
        const unsigned int run = ((n_list + kSelThreads - 1u) / kSelThreads) | 1u, first = threadIdx.x * run;
        for (unsigned int u0 = 0; u0 < run; u0 += kListAhead) {
          unsigned int rel[kListAhead];                // the adds are no memory accesses the compiler would read ahead of
#pragma unroll
          for (unsigned int u = 0; u < kListAhead; ++u)
            rel[u] = u0 + u < run && first + u0 + u < n_list ? sh.list[first + u0 + u] - v.lo : 0xffffffffu;
#pragma unroll
          for (unsigned int u = 0; u < kListAhead; ++u)
            if (rel[u] <= v.width) lds_add(base + 4u * (rel[u] >> shift), 1u);
        }
        lds_done();
        __syncthreads();
        const unsigned int mine = sh.hist[kLevelBins - 1 - threadIdx.x];
        sh.hist[kLevelBins - 1 - threadIdx.x] = 0u;
        unsigned int pk[3];
        pick_bin(mine, v.need, sh, pk);
        narrow(v, pk);
      }
      t = threshold_of(v);
      if (!alone) {                                  // those of the workgroups before this one
        unsigned int gt = 0u, eq = 0u;
#pragma unroll 4
        for (unsigned int i = threadIdx.x; i < list_before && i < n_list; i += kSelThreads) {
          const unsigned int k = sh.list[i];
          gt += k > t.T ? 1u : 0u;
          eq += (k == t.T && t.ties) ? 1u : 0u;
        }
        const unsigned int both = wave_sum((gt << 16) | eq);               // list_before <= 16384
        if (lane == 0) sh.wave[wave] = both;
        __syncthreads();
        const unsigned int sum = wave_sums(sh.wave, 0).total;
        gt_before += sum >> 16;
        eq_before = sum & 0xffffu;
      }
      break;
    }
  }
  if (threadIdx.x == 0) sh.failed = failed || outcome == kFailed ? 1u : 0u;
  __syncthreads();                                   // sh.off; sh.wave / sh.wave2 are free
  const lava_select_problem& out = a.p[opaque(prob)];   // read again here: fewer scalars live until now
  if (sh.failed != 0u) {                             // uniform over the problem's workgroups
    if (threadIdx.x < (unsigned)n_heads) out.head_counts[threadIdx.x] = -1;
    if (threadIdx.x <= (unsigned)n_heads) out.head_offsets[threadIdx.x] = 0;
    if (threadIdx.x == 0) st_dev(&st->error, 1u);
    if (threadIdx.x == 0 && out.error_dev != nullptr) *out.error_dev = 1;
    return;
  }
  const long long out_off = out.out_offset_dev ? (long long)*out.out_offset_dev : 0;
  write_survivors<KP>(key, rows, scores, wave_base, total, n_heads, t, gt_before, eq_before, kept_total, out.budget, alone,
                      bx == 0, sh, out.head_counts, out.head_offsets, out.kept_idx + out_off,
                      out.kept_scores ? out.kept_scores + out_off : nullptr);
}

// The same phases as separate launches (kernel boundaries take the place of the waits), for a problem
// too large to keep its whole grid resident.  STEP 0: first histogram and that of its end bins; 1..3: histograms of the
// interval's next 11 bits (nothing to do once it is decided); 4: counts; 5: write.  Digits of 11 bits because every launch
// counts: a bin of the first histogram (19 bits) and one of the ends (22) are one key wide after two of them; a prepared
// region has no histogram of the ends, and their 32 bits take the third.
constexpr int kStepBits = 11;
constexpr int kStepBins = 1 << kStepBits;
static_assert(next_hist_word(true) + 2 * kStepBins + (1 << (32 - 2 * kStepBits)) <= 3 * kSelBins &&
              next_hist_word(false) + 2 * kStepBins <= 3 * kSelBins && kEndShift <= 2 * kStepBits && kSelDigit0Shift <= 2 * kStepBits,
              "histogram area; two histograms behind one that was not prepared");
static_assert(kStepBins == 2 * kSelThreads && kStepBins <= (int)kListCap, "two bins per thread, counted in the list's place");

__device__ __forceinline__ unsigned int step_shift(const Interval& v) {
  return v.bits > (unsigned int)kStepBits ? v.bits - kStepBits : 0u;
}
// Bins an interval's next histogram has.
__device__ __forceinline__ int step_bins(const Interval& v) { return 1 << (v.bits - step_shift(v)); }

// The interval narrowed by histogram `h` (complete: an earlier launch's); thread t owns the bins
// kStepBins - 1 - 2 t and the one below.  Contains workgroup barriers.
__device__ __forceinline__ void step_narrow(Interval& v, const unsigned int* __restrict__ h, SelShared& sh) {
  const int n = step_bins(v), upper = kStepBins - 1 - 2 * (int)threadIdx.x;
  const unsigned int c1 = upper < n ? h[upper] : 0u, c0 = upper - 1 < n ? h[upper - 1] : 0u;
  unsigned int pair[3];
  pick_bin(c1 + c0, v.need, sh, pair);                // (pair's index, survivors needed from it, its count)
  // the pair's owner knows the two counts
  if (threadIdx.x == (unsigned int)(kLevelBins - 1) - pair[0]) {
    const bool in_upper = pair[1] <= c1;
    sh.before[0] = in_upper ? (unsigned int)upper : (unsigned int)(upper - 1);
    sh.before[1] = in_upper ? pair[1] : pair[1] - c1;
    sh.before[2] = in_upper ? c1 : c0;
  }
  __syncthreads();
  const unsigned int s = step_shift(v), skip = sh.before[0] << s, most = (1u << s) - 1u;
  v.lo += skip;
  v.width = v.width - skip < most ? v.width - skip : most;
  v.bits = s;
  v.need = sh.before[1];
  v.count = sh.before[2];
  __syncthreads();
}

template <int STEP, int KP>
__global__ void __launch_bounds__(kSelThreads) sel_step_kernel(const SelectBatch a) {
  const lava_select_problem pr = a.p[0];
  const int bx = (int)blockIdx.x, nb = (int)gridDim.x;
  unsigned int* hist = reinterpret_cast<unsigned int*>(a.ws + a.off_hist);
  unsigned int* step_hist = hist + next_hist_word(pr.primed != 0);
  unsigned int* blk = reinterpret_cast<unsigned int*>(a.ws + a.off_blk);
  const int64_t* __restrict__ seg_offsets = pr.seg_offsets;
  const int n_heads = a.n_heads;
  __shared__ SelShared sh;
  const int lane = threadIdx.x & 63, wave = sel_wave();
  const int total = (int)device_total(pr.total_entries, seg_offsets, n_heads);
  const int kept_total = (int)effective_budget(pr.budget, pr.budget_dev, total);
  const long long in_off = pr.in_offset_dev ? (long long)*pr.in_offset_dev : 0;
  const long long out_off = pr.out_offset_dev ? (long long)*pr.out_offset_dev : 0;
  const float* __restrict__ scores = pr.scores + in_off;
  if (STEP < 5 && kept_total == 0) return;
  const int wave_base = __builtin_amdgcn_readfirstlane((bx * kSelWaves + wave) * (64 * KP));
  Interval v = {0u, 0u, 0u, 0u, 0u};
  if (STEP >= 1 && kept_total > 0) {
    unsigned int pk[3];
    pick_bin(hist[kLevelBins - 1 - threadIdx.x], (unsigned int)kept_total, sh, pk);
    v = first_interval(pk);
    if (!pr.primed && v.bits == 32u && !decided(v))
      narrow_end(v, pk[0] == 0u, sh, [&](int w) { return hist[kLevelBins + w]; });
    __syncthreads();
    for (int l = 0; l < (STEP < 4 ? STEP - 1 : 3) && !decided(v); ++l) step_narrow(v, step_hist + l * kStepBins, sh);
    if (STEP <= 3 && decided(v)) return;
  }
  unsigned int key[KP];
  load_keys<KP>(scores, wave_base, total, key);
  if constexpr (STEP == 0) {
    sh.hist[threadIdx.x] = sh.list[threadIdx.x] = 0u;
    __syncthreads();
    count_first<KP>(key, sh.hist, sh.list);
    lds_done();
    __syncthreads();
    unsigned int c = sh.hist[threadIdx.x];
    if (threadIdx.x == 0) c -= missing<KP>(bx, total);
    if (c) __hip_atomic_fetch_add(&hist[threadIdx.x], c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const unsigned int of_end = sh.list[threadIdx.x];
    if (of_end) __hip_atomic_fetch_add(&hist[kLevelBins + threadIdx.x], of_end, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  } else if constexpr (STEP <= 3) {
    unsigned int* bins = sh.list;
    bins[threadIdx.x] = bins[threadIdx.x + kSelThreads] = 0u;
    __syncthreads();
    const unsigned int shift = step_shift(v), base = lds_offset(bins);
#pragma unroll
    for (int j = 0; j < KP; ++j) {
      const unsigned int rel = key[j] - v.lo;
      count_row(rel <= v.width, base + 4u * (rel >> shift));
    }
    lds_done();
    __syncthreads();
    for (int i = (int)threadIdx.x; i < step_bins(v); i += kSelThreads) {
      const unsigned int c = bins[i];
      if (c) __hip_atomic_fetch_add(&step_hist[(STEP - 1) * kStepBins + i], c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  } else {
    const Threshold t = kept_total > 0 ? threshold_of(v) : Threshold{0xffffffffu, 0u};
    if constexpr (STEP == 4) {
      unsigned int gt = 0u, eq = 0u;
#pragma unroll
      for (int j = 0; j < KP; ++j) {
        gt += (unsigned int)__popcll(__ballot(key[j] > t.T));
        eq += t.ties ? (unsigned int)__popcll(__ballot(key[j] == t.T)) : 0u;
      }
      if (lane == 0) { sh.wave[wave] = gt; sh.wave2[wave] = eq; }
      __syncthreads();
      gt = wave_sums(sh.wave, 0).total;
      eq = wave_sums(sh.wave2, 0).total;
      if (threadIdx.x == 0) { blk[bx] = gt; blk[nb + bx] = eq; }
    } else {
      unsigned int gt = 0u, eq = 0u;
      if (kept_total > 0)
        for (int b = (int)threadIdx.x; b < bx; b += kSelThreads) { gt += blk[b]; eq += blk[nb + b]; }
      gt = wave_sum(gt);
      eq = wave_sum(eq);
      if (lane == 0) { sh.wave[wave] = gt; sh.wave2[wave] = eq; }
      if (threadIdx.x <= n_heads)
        sh.off[threadIdx.x] = segment_start(seg_offsets, (int)threadIdx.x, n_heads, total);
      __syncthreads();
      gt = wave_sums(sh.wave, 0).total;
      eq = wave_sums(sh.wave2, 0).total;
      __syncthreads();
      write_survivors<KP>(key, 0xffffffffu, scores, wave_base, total, n_heads, t, gt, eq, kept_total, pr.budget, false, bx == 0,
                                 sh, pr.head_counts, pr.head_offsets, pr.kept_idx + out_off,
                                 pr.kept_scores ? pr.kept_scores + out_off : nullptr);
    }
  }
}

// Workgroups of the fused kernel that can be resident at once on the current device.
static int fused_capacity() {
  static int cached[64];
  static bool known[64];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 0;
  if (!known[dev]) {
    int per_cu = 0, cus = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, sel_fused_kernel<kMostKeys>, kSelThreads, 0) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
      return 0;
    cached[dev] = per_cu * cus;
    known[dev] = true;
  }
  return cached[dev];
}

// Keys per lane for a launch that starts with problems[0 .. n - 1], of whose workgroups `cap` may be resident:
// few, because every row of keys costs 0.3 us in all, until the number of workgroups that exchange their
// counts costs more.  In-kernel times, not prepared, in us (workgroups): 33 K entries: 2 keys 11.0 (17),
// 4 keys 11.9 (9), 8 keys 13.3 (5); 48 K: 11.9 (24), 12.4 (12); 262 K: 17.7 (128), 16.0 (64), 15.8 (32),
// 16 keys 18.8 (16).  Calls, 1 M entries, budget n/100 and n/4: 8 keys 25.8 and 30.3 (128), 12 keys 25.5 and 31.8 (86);
// 1.5 M: 8 keys 28.5 and 35.6 (184), 12 keys 27.4 and 35.6 (123), 16 keys 28.6 and 39.4 (92).
static int fused_keys(const lava_select_problem* problems, int n, int cap) {
  for (int keys : {2, 4, 8}) {
    int64_t sum = 0, widest = 0;
    for (int i = 0; i < n; ++i) {
      const int64_t nb = workgroups_for(problems[i].total_entries, keys);
      sum += nb;
      if (nb > widest) widest = nb;
    }
    if (sum <= cap && widest <= (keys == 2 ? 20 : keys == 4 ? 64 : 128)) return keys;
  }
  return kMostKeys;
}

// Calls f(std::integral_constant<int, KP>) for a number of keys per lane fused_keys returned.
template <class F>
static void with_keys(int keys, F&& f) {
  switch (keys) {
    case 2: f(std::integral_constant<int, 2>{}); break;
    case 4: f(std::integral_constant<int, 4>{}); break;
    case 8: f(std::integral_constant<int, 8>{}); break;
    default: f(std::integral_constant<int, kMostKeys>{}); break;
  }
}

// Selections of a batch: consecutive problems are packed into launches of the fused kernel as long
// as their workgroups fit into half of the device together (they all have to be resident: the workgroups
// of a problem wait for each other; should another stream hold compute units for so long that
// a bounded wait gives up, the kernel marks the outputs and the status call reports it).  A single
// problem wider than that runs as step launches.
int32_t launch_select_batch(int n_heads, int n_problems, const lava_select_problem* problems, int64_t max_total,
                            void* ws, hipStream_t s, bool cleared) {
  const SelectWorkspace w = make_select_workspace(max_total);
  SelectBatch a;
  a.n_heads = n_heads;
  a.ws_stride = w.bytes;
  a.off_hist = w.off_hist;
  a.off_state = w.off_state;
  a.off_blk = w.off_blk;
  const dim3 block(kSelThreads);
  a.spin_limit = tuning().barrier_spin_limit > 0 ? (unsigned int)tuning().barrier_spin_limit : kSpinLimit;
  // Half of what the device can keep resident: the waits need every workgroup of a launch on the device
  // at once, and the margin leaves room for whatever else is running there.
  const int cap = fused_capacity() / 2 < kFusedMaxBlocks ? fused_capacity() / 2 : kFusedMaxBlocks;
  int first = 0, group_end = 0, keys = kMostKeys;
  while (first < n_problems) {
    if (first == group_end) {
      // the next group of at most kMaxSelProblems problems: one choice of keys per lane, one clearing launch
      const int n = n_problems - first < kMaxSelProblems ? n_problems - first : kMaxSelProblems;
      group_end = first + n;
      keys = fused_keys(problems + first, n, cap);
      // Regions and survivor counts are cleared unless no kernel of the group needs that: the one-launch
      // selection of a problem that fits one workgroup does not, and that of a prepared one clears its counts itself.
      bool needed = false;
      a.primed_mask = 0u;
      for (int i = 0; i < n; ++i) {
        const lava_select_problem& pr = problems[first + i];
        a.p[i] = pr;
        if (pr.primed) a.primed_mask |= 1u << i;
        const int64_t nb = workgroups_for(pr.total_entries, keys);
        if (nb > cap || (nb > 1 && !pr.primed)) needed = true;
      }
      if (needed && !cleared) {
        a.ws = static_cast<char*>(ws) + (size_t)first * w.bytes;
        ProfScope ps(KID_SEL_INIT, s);
        hipLaunchKernelGGL(sel_init_kernel, dim3(n), block, 0, s, a);
      }
    }
    int count = 0;
    int64_t blocks = 0, widest = 1;
    a.primed_mask = 0u;
    while (first + count < group_end) {
      const lava_select_problem& pr = problems[first + count];
      const int64_t nb = workgroups_for(pr.total_entries, keys);
      if (count > 0 && blocks + nb > cap) break;
      a.first_block[count] = (int)blocks;
      blocks += nb;
      if (nb > widest) widest = nb;
      a.p[count] = pr;
      if (pr.primed) a.primed_mask |= 1u << count;
      ++count;
    }
    a.n_problems = count;
    a.first_block[count] = (int)blocks;
    a.seg_words = segment_words(keys, widest, w.blk_words);
    a.ws = static_cast<char*>(ws) + (size_t)first * w.bytes;
    const bool fused = blocks <= cap;
    if (fused) {
      ProfScope ps(KID_SEL_FUSED, s);
      const dim3 grid((unsigned)blocks);
      with_keys(keys, [&](auto kp) { hipLaunchKernelGGL(sel_fused_kernel<decltype(kp)::value>, grid, block, 0, s, a); });
    } else {                                               // a single problem wider than the device allows
      ProfScope ps(KID_SEL_STEPS, s);
      // Keys per lane: 32, which read a problem in few workgroups, where those still fill three quarters of the device's
      // compute units, else 16 (budget n/100 and n/4, us: 4 M 49.5 and 56.7 with 32, 44.3 and 48.6 with 16; 8 M, prepared,
      // 48.7 and 63.4, 49.5 and 66.0; 16 M within 2 % of each other 118 and 131, 132 and 144).
      const int64_t total = a.p[0].total_entries;
      const bool wide = workgroups_for(total, 32) * 4 >= 3 * (int64_t)sweep_device_wgs();
      auto steps = [&](auto kp) {
        constexpr int KP = decltype(kp)::value;
        const dim3 grid((unsigned)workgroups_for(total, KP));
        if (!a.p[0].primed) hipLaunchKernelGGL((sel_step_kernel<0, KP>), grid, block, 0, s, a);
        hipLaunchKernelGGL((sel_step_kernel<1, KP>), grid, block, 0, s, a);
        hipLaunchKernelGGL((sel_step_kernel<2, KP>), grid, block, 0, s, a);
        if (a.p[0].primed) hipLaunchKernelGGL((sel_step_kernel<3, KP>), grid, block, 0, s, a);   // its end bins are 32 bits wide
        hipLaunchKernelGGL((sel_step_kernel<4, KP>), grid, block, 0, s, a);
        hipLaunchKernelGGL((sel_step_kernel<5, KP>), grid, block, 0, s, a);
      };
      if (wide) steps(std::integral_constant<int, 32>{});
      else steps(std::integral_constant<int, 16>{});
    }
    const int32_t st = launch_status();
    if (st != LAVA_OK) return st;
    first += count;
  }
  return LAVA_OK;
}

int32_t launch_select(int n_heads, const float* scores, const int64_t* seg_offsets, int64_t total,
                      int64_t budget, const int64_t* budget_dev, int32_t* head_counts,
                      int64_t* head_offsets, int32_t* kept_idx, float* kept_scores, void* ws,
                      hipStream_t s) {
  lava_select_problem pr;
  pr.scores = scores;
  pr.seg_offsets = seg_offsets;
  pr.total_entries = total;
  pr.budget = budget;
  pr.budget_dev = budget_dev;
  pr.head_counts = head_counts;
  pr.head_offsets = head_offsets;
  pr.kept_idx = kept_idx;
  pr.kept_scores = kept_scores;
  pr.in_offset_dev = nullptr;
  pr.out_offset_dev = nullptr;
  pr.error_dev = nullptr;
  pr.primed = 0;
  return launch_select_batch(n_heads, 1, &pr, total, ws, s);
}

// Error words of the first n_problems regions laid out for max_total: flag = OR of them.
int32_t select_error_flag(const void* ws, int64_t max_total, int n_problems, hipStream_t s, int* flag) {
  const SelectWorkspace w = make_select_workspace(max_total);
  *flag = 0;
  for (int p = 0; p < n_problems; ++p) {
    const SelectState* st = reinterpret_cast<const SelectState*>(static_cast<const char*>(ws) + (size_t)p * w.bytes +
                                                                 w.off_state);
    unsigned int host = 0u;
    if (hipMemcpyAsync(&host, &st->error, sizeof(host), hipMemcpyDeviceToHost, s) != hipSuccess) return LAVA_ERR_HIP;
    if (hipStreamSynchronize(s) != hipSuccess) return LAVA_ERR_HIP;
    *flag |= (int)host;
  }
  return LAVA_OK;
}

}  // namespace lava

// ------------------------------------------------------------------------------------------
// lava_select_topk for callers that cannot allocate (code under HIP graph capture, serving loops
// and harnesses that forbid hipMalloc): the selection's workspace is a fixed array in the
// library's own device image instead of a caller buffer.  Every GPU holds its own copy of the
// array at its own address; the address is looked up once per device and the kernels receive it
// as an ordinary pointer argument, exactly as they receive a caller's workspace.
// ------------------------------------------------------------------------------------------
namespace {
constexpr int64_t kStaticMaxEntries = LAVA_SELECT_STATIC_MAX_ENTRIES;
constexpr size_t kStaticScratchBytes = lava::select_layout(kStaticMaxEntries).bytes;
static_assert(kStaticScratchBytes <= ((size_t)2 << 20), "the built-in scratch array is meant to stay small");
}  // namespace

static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

namespace {
constexpr int kMaxDevices = 64;
void* g_scratch_ptr[kMaxDevices];       // device address of `scratch` on each GPU, once known
bool g_scratch_known[kMaxDevices];

// Device address of this GPU's copy of the array (the array's name is a host-side handle, never a
// device address).
int32_t scratch_of_current_device(void** out) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return LAVA_ERR_HIP;
  if (!g_scratch_known[dev]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || p == nullptr) return LAVA_ERR_HIP;
    g_scratch_ptr[dev] = p;
    g_scratch_known[dev] = true;
  }
  *out = g_scratch_ptr[dev];
  return LAVA_OK;
}
}  // namespace

extern "C" int32_t lava_select_topk_static(int32_t n_heads, const float* scores, const int64_t* seg_offsets,
                                           int64_t total_entries, int64_t budget, const int64_t* budget_dev,
                                           int32_t* head_counts, int64_t* head_offsets, int32_t* kept_idx,
                                           float* kept_scores, void* hip_stream) {
  if (n_heads < 1) return LAVA_ERR_INVALID_ARG;
  if (n_heads > lava::kMaxHeads) return LAVA_ERR_SHAPE;
  const lava_select_problem p = {scores,      seg_offsets,  total_entries, budget,     budget_dev,
                                 head_counts, head_offsets, kept_idx,      kept_scores, nullptr, nullptr, nullptr, 0};
  const int32_t st = lava::check_select_problem(n_heads, p);
  if (st != LAVA_OK) return st;
  if (total_entries > kStaticMaxEntries) return LAVA_ERR_WORKSPACE;   // beyond what the built-in array holds
  void* ws = nullptr;
  const int32_t sw = scratch_of_current_device(&ws);
  if (sw != LAVA_OK) return sw;
  lava::discard_stale_error();
  // histograms, barrier counter and error word are cleared by the selection's own first kernel
  return lava::launch_select_batch(n_heads, 1, &p, total_entries, ws, static_cast<hipStream_t>(hip_stream));
}

