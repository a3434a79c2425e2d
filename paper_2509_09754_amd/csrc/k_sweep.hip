// The three sweeps over a layer's cache (Def. 1 / Eq. 3 with the attention rows of Sec. 2):
//
//   vnorm   V once:  per-row L1 norms, per-workgroup maxima                 -> Vbar (Thm. 1)
//   stats   K once:  logits of the w window rows against every key on the matrix cores, online
//                    row max / row sum per workgroup                        -> softmax normaliser
//   scores  K again: the same logits, exp2 against the merged normaliser, mean over the window
//                    rows, max over the query heads of the KV group (Sec. 4.3)
//
// The window product is the one dense contraction of the path: per KV head a
// [G*w] x d_h x N GEMM.  Each wavefront owns 32-key tiles.  A tile travels HBM -> LDS with
// coalesced 128-bit direct-to-LDS loads (no staging registers) into a wavefront-private ring of
// XOR-swizzled buffers, several tiles ahead of the one being multiplied; it is then read in MFMA
// operand layout and multiplied against the group's query rows, which stay in registers for the
// whole sweep.  The ring is private to the wavefront, so the sweep needs no workgroup barrier:
// arrival of a tile is a vmcnt wait that leaves the younger tiles in flight.
//
// MFMA 32x32 layouts used below (wave64): operand lane l supplies row/column l%32 and k-slice
// l/32; result register v of lane l is element (8*(v/4) + 4*(l/32) + v%4, l%32).
//   stats  : D = K_tile * Q^T  -> a lane holds 16 keys of ONE query row: row reductions stay in-lane
//   scores : D = Q * K_tile^T  -> a lane holds 16 query rows of ONE key: the window mean stays in-lane
#include <math.h>

#include "budget_wave.h"
#include "common.h"
#include "tile_ring.h"
#include "xblock.h"

namespace lava {

// "last workgroup done" tickets in the workspace (zeroed by the first kernel of every call)
constexpr int kCounterPool = 0;                         // poolstat: one two-level ticket
// control words of the persistent sweep, behind the ticket (a sequence's counter region)
constexpr int kCtlError = kArriveWords;                 // a wait for other workgroups gave up (first sequence's region)
constexpr int kCtlDoneA = kArriveWords + 1;             // [64] statistics units completed, per KV head of the sequence
constexpr int kCtlUnitA = kCtlDoneA + 64;               // [H_kv * blocks_x] claim word of every statistics unit of the sequence

// Wavefronts per workgroup and ring depth.  Kernels whose registers fit twice into a SIMD come in two
// shapes.  Wide (W = 8): 8 wavefronts (2 per SIMD: one wavefront's exponentials overlap the
// other's MFMAs and waits), a 128 KiB ring, so a CU holds one workgroup: the shape for a launch
// whose workgroups all start together (one sequence).  Narrow (W = 4): 4 wavefronts and a 64 KiB
// ring, two workgroups per CU with the same registers, wavefronts and bytes in flight per CU: in a
// launch of several rounds of workgroups (a batch) the two run out of phase, and one's set-up and
// tail hide behind the other's streaming.  The f32 / d_h 128 kernels need more than 256 registers:
// 4 wavefronts and the whole ring in either case.
constexpr int kFusedTilesWide = 128;
constexpr int kFusedTilesNarrow = 96;
template <int DT, int D, int W>
struct Shape {
  static_assert(W == 4 || W == 8, "wavefronts per workgroup");
  static constexpr bool kBig = DT == LAVA_F32 && D == 128;
  static constexpr bool kNarrow = W == 4 && !kBig;
  static constexpr int kWaves = kBig ? 4 : W;
  static constexpr int kThreads = kWaves * 64;
  static constexpr int kMinWaves = kNarrow ? 2 : 1;      // per SIMD, for the register allocator
  static constexpr int kRingBytes = kNarrow ? 64 * 1024 : 128 * 1024;
  static constexpr int kStagesRaw = kRingBytes / (kWaves * Tile<DT, D>::kTileBytes);
  static constexpr int kStages = kStagesRaw > 4 ? 4 : kStagesRaw;
  static constexpr int kFusedTiles = kNarrow ? kFusedTilesNarrow : kFusedTilesWide;   // span of raw scores kept in LDS
  static_assert(kStages >= 2 && kStages <= kMaxRingStages, "ring depth");
};

// Sum over the wavefront's lanes in a fixed order, in every lane: data-parallel-primitive moves (shifts inside rows
// of 16 lanes, then the last lane of one row to the next ones) instead of 24 trips through the LDS unit.
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_add_f64(double x) {
  const unsigned long long b = (unsigned long long)__double_as_longlong(x);
  const unsigned int lo = (unsigned int)__builtin_amdgcn_update_dpp(0, (int)(unsigned int)b, CTRL, ROWS, 0xf, false);
  const unsigned int hi = (unsigned int)__builtin_amdgcn_update_dpp(0, (int)(unsigned int)(b >> 32), CTRL, ROWS, 0xf, false);
  return x + __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));   // +0 where no lane shifts in
}
__device__ __forceinline__ double wave_sum_f64(double x) {
  x = dpp_add_f64<0x111, 0xf>(x);
  x = dpp_add_f64<0x112, 0xf>(x);
  x = dpp_add_f64<0x114, 0xf>(x);
  x = dpp_add_f64<0x118, 0xf>(x);
  x = dpp_add_f64<0x142, 0xa>(x);
  x = dpp_add_f64<0x143, 0xc>(x);
  const unsigned long long b = (unsigned long long)__double_as_longlong(x);
  const unsigned int lo = (unsigned int)__builtin_amdgcn_readlane((int)(unsigned int)b, 63);
  const unsigned int hi = (unsigned int)__builtin_amdgcn_readlane((int)(unsigned int)(b >> 32), 63);
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// Maximum over the wavefront's lanes, in every lane, of values that are not negative.
template <int CTRL, int ROWS>
__device__ __forceinline__ float dpp_max_f32(float x) {
  return fmaxf(x, __uint_as_float((unsigned int)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(x), CTRL, ROWS, 0xf, false)));
}
__device__ __forceinline__ float wave_max_f32(float x) {
  x = dpp_max_f32<0x111, 0xf>(x);
  x = dpp_max_f32<0x112, 0xf>(x);
  x = dpp_max_f32<0x114, 0xf>(x);
  x = dpp_max_f32<0x118, 0xf>(x);
  x = dpp_max_f32<0x142, 0xa>(x);
  x = dpp_max_f32<0x143, 0xc>(x);
  return __uint_as_float((unsigned int)__builtin_amdgcn_readlane((int)__float_as_uint(x), 63));
}

// Layer statistic from per-lane partial sums S = sum s, T = sum s ln s (fp64): fixed-order reduction
// over lanes, wavefronts and, by the last workgroup to arrive, workgroups; then
// e = (ln S - T / S) / n_entries  (Eq. 4-5 in closed form).  Contains workgroup barriers.  Returns true in
// every thread of that last workgroup, whose thread 0 has then also left the statistic (as stored,
// rounded to fp32) in s_t[0] for whatever the workgroup does next with it (not yet published by a barrier).
template <int THREADS>
__device__ __forceinline__ bool entropy_finish(double acc_s, double acc_t, double2* __restrict__ ent_part,
                                               uint32_t* __restrict__ counters, unsigned int n_blocks,
                                               unsigned int block_id, double n_entries,
                                               float* __restrict__ layer_stat, double* s_s, double* s_t,
                                               unsigned int* s_last, const uint32_t* error_word = nullptr) {
  constexpr int kW = THREADS / 64;
  acc_s = wave_sum_f64(acc_s);
  acc_t = wave_sum_f64(acc_t);
  if ((threadIdx.x & 63) == 0) { s_s[threadIdx.x >> 6] = acc_s; s_t[threadIdx.x >> 6] = acc_t; }
  __syncthreads();
  if (threadIdx.x == 0) {
    double S = 0.0, Tt = 0.0;
    for (int i = 0; i < kW; ++i) { S += s_s[i]; Tt += s_t[i]; }
    double2* mine = &ent_part[block_id];
    st_dev_f64(&mine->x, S);
    st_dev_f64(&mine->y, Tt);
  }
  if (!arrive_last(&counters[kCounterPool], n_blocks, block_id, s_last)) return false;
  // last workgroup: thread t sums partials t, t + THREADS, ... then the same fixed tree as above
  double S = 0.0, Tt = 0.0;
  for (unsigned int i = threadIdx.x; i < n_blocks; i += THREADS) {
    S += ld_dev_f64(&ent_part[i].x);
    Tt += ld_dev_f64(&ent_part[i].y);
  }
  S = wave_sum_f64(S);
  Tt = wave_sum_f64(Tt);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) { s_s[threadIdx.x >> 6] = S; s_t[threadIdx.x >> 6] = Tt; }
  __syncthreads();
  if (threadIdx.x != 0) return true;
  S = 0.0; Tt = 0.0;
  for (int i = 0; i < kW; ++i) { S += s_s[i]; Tt += s_t[i]; }
  double e = 0.0;
  if (S > 0.0) e = (log(S) - Tt / S) / n_entries;
  if (error_word != nullptr && ld_dev(error_word) != 0u) e = (double)NAN;   // scores of this call are not to be used
  layer_stat[0] = (float)e;
  s_t[0] = (double)(float)e;
  return true;
}

// What the budget rule reads, fetched by the lanes of wavefront 0 well before the statistic exists (any
// workgroup may turn out to be the one that forms it; the loads are few and hit in L2): layers lane and
// lane + 64 of sequence b's rows.
struct PlanInputs {
  long long lo[2], hi[2], total;
  float e[2];
};
static_assert(kMaxPlannedLayers <= 128, "two layers per lane");
__device__ __forceinline__ PlanInputs plan_prefetch(const BudgetPlanArgs& plan, int b) {
  PlanInputs in = {};
  if (plan.e == nullptr || threadIdx.x >= 64) return in;
  const long long row = (long long)b * plan.n_layers;
  in.total = (long long)plan.total[b];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int i = (int)threadIdx.x + 64 * j;
    if (i < plan.n_layers) {
      in.lo[j] = (long long)plan.lo[row + i];
      in.hi[j] = (long long)plan.hi[row + i];
      if (i != plan.layer) in.e[j] = plan.e[row + i];
    }
  }
  return in;
}

// Budgets of sequence b of the batch from the statistics of its layers (Alg. 2, inner loop), by
// wavefront 0 of the workgroup that has just formed the statistic e_new of layer plan.layer: the same
// routine, on the same values, as the budgets kernel.  `lds`: sizeof(BudgetScratchT<kMaxPlannedLayers>)
// bytes, 8-aligned, that no other wavefront of the workgroup touches meanwhile.  A NaN statistic (a
// failed launch) leaves all budgets of the sequence at -1.
__device__ __forceinline__ void plan_budgets(const BudgetPlanArgs& plan, const PlanInputs& in, int b, float e_new,
                                             void* lds) {
  if (threadIdx.x >= 64) return;
  using Scratch = BudgetScratchT<kMaxPlannedLayers>;
  Scratch* sc = static_cast<Scratch*>(lds);
  const int lane = (int)threadIdx.x, n = plan.n_layers;
  const long long row = (long long)b * n;
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int i = lane + 64 * j;
    if (i < n) {
      sc->ed[i] = i == plan.layer ? (double)e_new : (double)in.e[j];
      sc->lo[i] = in.lo[j];
      sc->hi[i] = in.hi[j];
    }
  }
  if (lane == 0) plan.e[row + plan.layer] = e_new;
  WaveSync::sync();
  long long* out_b = reinterpret_cast<long long*>(plan.out) + row;
  int bad = e_new != e_new ? 1 : 0;
  if (n == 1) {
    // a single layer takes the whole total (its quota is total * e / e, exactly), if the bounds allow it:
    // what the rule below returns, without its reductions across the wavefront
    const long long lo0 = __shfl(in.lo[0], 0), hi0 = __shfl(in.hi[0], 0);
    if (lane == 0) out_b[0] = (!bad && lo0 >= 0 && lo0 <= in.total && in.total <= hi0) ? in.total : -1;
    return;
  }
  if (!bad)
    bad = allocate_budgets_wave<WaveSync>(lane, n, sc->ed, in.total, sc->lo, sc->hi, out_b, sc->quota, sc->base,
                                          sc->freel, sc->frac, sc->state);
  if (bad)
    for (int i = lane; i < n; i += 64) out_b[i] = -1;
}

// One tile of keys (its fragments in kf) into a wavefront's running statistics: per head of the chunk this lane's
// maximum of the raw dot products of its query row (lane % 32) and the sum of exp2((dot - max) * c2) over the keys it
// has seen (the two lane halves see different keys of the same rows).
template <int DT, int D, int GT>
__device__ __forceinline__ void stats_tile(const u32x4 (&kf)[Tile<DT, D>::kSteps], long long tile, long long n, const RowMap& rm,
                                           float c2, const u32x4 (&qf)[GT][kQVec<DT, D>], bool q_parts, int lane,
                                           float (&m_run)[GT], float (&z_run)[GT]) {
  const int r = lane & (rm.rph - 1), half = lane >> 5, w = rm.w;   // r: window row, in the first block of two
  const long long key0 = tile * kTileKeys;
  // 32-bit inputs: all heads' products at once (the split of the keys is shared); bf16: head by head, so that
  // the next head's matrix instructions run beside this head's exponentials
  f32x16 all[DT == LAVA_F32 ? GT : 1];
  if constexpr (DT == LAVA_F32) dot_tiles<D, GT, true>(kf, qf, q_parts, all);
  auto head_dots = [&](int t) -> f32x16 {
    if constexpr (DT == LAVA_F32) return all[t];
    else return dot_tile<D, true>(kf, qf[t]);
  };
  if (key0 + kTileKeys - 1 <= n - w) {
    // every row sees every key of the tile: straight-line code
    f32x16 acc = head_dots(0);
#pragma unroll
    for (int t = 0; t < GT; ++t) {
      f32x16 nxt = acc;
      if (t + 1 < GT) nxt = head_dots(t + 1);
      float tmax = fmaxf(acc[0], acc[1]);
#pragma unroll
      for (int v = 2; v < 16; ++v) tmax = fmaxf(tmax, acc[v]);
      const float mn = fmaxf(m_run[t], tmax);
      const float mc = mn * c2;
      float zs = 0.0f;
#pragma unroll
      for (int v = 0; v < 16; ++v) zs += fast_exp2(fmaf(acc[v], c2, -mc));
      z_run[t] = z_run[t] * fast_exp2((m_run[t] - mn) * c2) + zs;   // exp2(-inf) = 0 on the first tile
      m_run[t] = mn;
      acc = nxt;
    }
  } else {
    // tile touches the window or the end of the sequence: mask what a row may not see
    const int rel0 = (int)(key0 - (n - w));                // position of the tile's first key relative to N - w
#pragma unroll
    for (int t = 0; t < GT; ++t) {
      // window row of this lane in block t (a chunk starts at an even block when heads have two blocks);
      // row rr sees relative positions <= min(rr, w - 1)
      const int rr = r + ((rm.bph == 2 && (t & 1)) ? 32 : 0);
      const int row_limit = rr < w - 1 ? rr : w - 1;
      f32x16 acc = head_dots(t);
#pragma unroll
      for (int v = 0; v < 16; ++v)
        if (rel0 + 8 * (v / 4) + 4 * half + (v % 4) > row_limit) acc[v] = -INFINITY;
      float tmax = acc[0];
#pragma unroll
      for (int v = 1; v < 16; ++v) tmax = fmaxf(tmax, acc[v]);
      if (tmax > -INFINITY) {
        const float mn = fmaxf(m_run[t], tmax);
        const float mc = mn * c2;
        float zs = 0.0f;
#pragma unroll
        for (int v = 0; v < 16; ++v) zs += fast_exp2(fmaf(acc[v], c2, -mc));
        const float f = (m_run[t] == mn) ? 1.0f : fast_exp2((m_run[t] - mn) * c2);
        z_run[t] = z_run[t] * f + zs;
        m_run[t] = mn;
      }
    }
  }
}

// The statistics sweep of one wavefront: tiles first, first + WAVES, ... (cnt of them) of the head
// at kg, whose first STAGES - 1 tiles have already been requested into `ring`.  The assignment of tiles to
// wavefronts is static: the sums depend on the order, and results must not depend on timing.  Tile `it` sits in ring
// slot (it + slot0) % STAGES (slot0 != 0 when another sweep of the same wavefront used the ring just before and
// requested these tiles).
template <int DT, int D, int GT, int WAVES, int STAGES>
__device__ __forceinline__ void stats_tiles(const TileDma<DT, D>& dma, const FragReader<DT, D>& frags,
                                            const char* __restrict__ kg, long long n, const RowMap& rm, float c2,
                                            long long first, int cnt, u32x4* ring,
                                            const u32x4 (&qf)[GT][kQVec<DT, D>], bool q_parts, int lane,
                                            float (&m_run)[GT], float (&z_run)[GT], int slot0 = 0) {
  using T = Tile<DT, D>;
  static_assert((STAGES & (STAGES - 1)) == 0, "ring slots are taken modulo a power of two");
#pragma unroll
  for (int t = 0; t < GT; ++t) { m_run[t] = -INFINITY; z_run[t] = 0.0f; }
  const unsigned int ring_addr = lds_addr(ring);
  for (int it = 0; it < cnt; ++it) {
    const int ahead = it + STAGES - 1;
    if (ahead < cnt)
      dma.issue(kg, first + (long long)ahead * WAVES, n, lane, ring + ((ahead + slot0) % STAGES) * T::kTileChunks);
    const int younger = cnt - 1 - it < STAGES - 1 ? cnt - 1 - it : STAGES - 1;
    wait_tile<DT, D>(younger);
    u32x4 kf[T::kSteps];
    frags.read(ring_addr + ((it + slot0) % STAGES) * T::kTileBytes, kf);
    stats_tile<DT, D, GT>(kf, first + (long long)it * WAVES, n, rm, c2, qf, q_parts, lane, m_run, z_run);
  }
}

// Merge of the two lane halves (same row, different keys), then of a chunk's wavefronts in wavefront order.
// Thread (head * 32 + row) of the workgroup, heads counted through its NC chunks, returns true and the merged
// (max, sum) of its row.  Contains a workgroup barrier.
template <int GT, int WAVES, int NC>
__device__ __forceinline__ bool stats_merge_waves(float (&m_run)[GT], float (&z_run)[GT], float c2, int lane, int wave,
                                                  float2 (*s_red)[kMaxChunkHeads * 32], float2& out) {
  const int r = lane & 31, half = lane >> 5;
#pragma unroll
  for (int t = 0; t < GT; ++t) {
    const float m2 = __shfl_xor(m_run[t], 32);
    const float z2 = __shfl_xor(z_run[t], 32);
    merge_stat(m_run[t], z_run[t], m2, z2, c2);
    if (half == 0) s_red[wave][t * 32 + r] = make_float2(m_run[t], z_run[t]);
  }
  __syncthreads();
  constexpr int kPerChunk = WAVES / NC;                      // wavefronts of a chunk
  static_assert(NC * GT <= WAVES * 2, "a thread per row");
  if (threadIdx.x >= NC * GT * 32) return false;
  const int first_wave = NC == 1 ? 0 : (int)(threadIdx.x / (GT * 32)) * kPerChunk, row = (int)(threadIdx.x % (GT * 32));
  float2 p[kPerChunk];
#pragma unroll
  for (int wv = 0; wv < kPerChunk; ++wv) p[wv] = s_red[first_wave + wv][row];
  float m = -INFINITY, z = 0.0f;
  merge_stats<kPerChunk>(p, c2, m, z);
  out = make_float2(m, z);
  return true;
}

// sum of |x| over 16 bytes, added to s
template <int DT>
__device__ __forceinline__ float abs_sum16(const u32x4& x, float s) {
  const unsigned int u[4] = {x.x, x.y, x.z, x.w};
  if constexpr (DT == LAVA_BF16) {
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    const bf16x2 ones = {(__bf16)1.0f, (__bf16)1.0f};
#pragma unroll
    for (int i = 0; i < 4; ++i)   // clear both sign bits, then a.x * 1 + a.y * 1 + s in one instruction
      s = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, u[i] & 0x7fff7fffu), ones, s, false);
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i) s += fabsf(__uint_as_float(u[i]));
  }
  return s;
}

// The selection region a primed call prepares for sequence z of the launch: histograms and state to zero
// (the score kernels of the same call then fill the first histogram).  Called by one workgroup.
__device__ __forceinline__ void clear_selection_region(const SweepArgs& a, int z, int threads) {
  if (a.sel_ws == nullptr) return;
  char* region = a.sel_ws + (size_t)(a.first_seq + z) * a.sel_stride;
  unsigned int* hist = reinterpret_cast<unsigned int*>(region + a.sel_off_hist);
  unsigned int* state = reinterpret_cast<unsigned int*>(region + a.sel_off_state);
  for (int i = threadIdx.x; i < 3 * kSelBins; i += threads) hist[i] = 0u;
  if (threadIdx.x < kSelStateWords) state[threadIdx.x] = 0u;
}

// A group split into chunks: the raw scores of head g's span of tiles start from +0 (the chunks' workgroups join
// theirs with an integer maximum).  Done by the first kernel of the call; as a launch of its own it took 4.7 us.
// Called after the tile loop: the ring counts loads, which stores in between would upset.
__device__ __forceinline__ void clear_raw_scores(const SweepArgs& a, const SweepSeq& sq, int g, long long t_begin, long long t_end,
                                                 int threads) {
  if (a.n_chunks == 1) return;
  const long long n_prefix = sq.n - a.w;
  float* raw = reinterpret_cast<float*>(a.ws + sq.ws_off + a.off_sraw) + (long long)g * n_prefix;
  long long end = t_end * kTileKeys;
  if (end > n_prefix) end = n_prefix;
  for (long long i = t_begin * kTileKeys + threadIdx.x; i < end; i += threads) raw[i] = 0.0f;
}

// Workgroup barrier that leaves the tile loads in flight (what it orders is the reads and loads of the asm and
// DMA protocol above, each of which has waited for its own).
__device__ __forceinline__ void wave_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// A statistics / scores launch numbers the workgroups of all its sequences through (SweepSeq::unit_base): sequence
// z of the launch, KV head and chunk y, span x.  A grid as wide as the longest sequence left the dispatcher to
// start and retire the missing workgroups of the others: 16 sequences of 4096 to 65536 tokens, 3200 workgroups
// of which 1992 had work, 4.3 us between two of them on a slot where a full grid has 1.
struct Unit {
  int z, y, x;
};
__device__ __forceinline__ RowMap row_map(const SweepArgs& a) { return RowMap{a.heads, a.G, a.bph, a.rph, a.w}; }
__device__ __forceinline__ Unit unit_of_block(const SweepArgs& a) {
  Unit u;
  u.z = 0;
  if (a.n_seq > 1) {
    const int lane = threadIdx.x & 63;
    const unsigned long long at = __ballot(lane < a.n_seq && a.s[lane < a.n_seq ? lane : 0].unit_base <= (int)blockIdx.x);
    u.z = 63 - __builtin_clzll(at);                            // unit_base[0] = 0
  }
  const unsigned int rel = blockIdx.x - (unsigned int)a.s[u.z].unit_base, bx = (unsigned int)a.s[u.z].blocks_x;
  u.y = __builtin_amdgcn_readfirstlane((int)(rel / bx));
  u.x = (int)rel - u.y * (int)bx;
  return u;
}
static_assert(kMaxSeqPerLaunch <= 64, "one lane per sequence");

// The value-norm sweep of one wavefront: tiles first, first + WAVES, ... (cnt of them) of the head at
// vg, whose first STAGES - 1 tiles have already been requested into `ring`.  Returns this lane's maximum
// over its rows (row lane % 32 of every tile) of sum_c |V[row, c]|; with token_norm the rows' own norms
// also go to row_norm (indexed by position).  CHAIN > 0: as the ring drains, the first STAGES - 1 of the tiles
// next_first, next_first + CHAIN, ... (next_cnt of them) at `next` (the head's keys) are requested into the slots
// that follow, so that the statistics sweep continues without a gap: its tile `it` is in slot (cnt + it) % STAGES.
template <int DT, int D, int WAVES, int STAGES, int CHAIN>
__device__ __forceinline__ float vnorm_tiles(const TileDma<DT, D>& dma, const FragReader<DT, D>& frags,
                                             const char* __restrict__ vg, const char* __restrict__ next, long long n,
                                             long long first, int cnt, long long next_first, int next_cnt, u32x4* ring,
                                             int lane, bool token_norm, float* __restrict__ row_norm) {
  using T = Tile<DT, D>;
  static_assert((STAGES & (STAGES - 1)) == 0, "ring slots are taken modulo a power of two");
  const unsigned int ring_addr = lds_addr(ring);
  const int total = CHAIN > 0 ? cnt + next_cnt : cnt;        // tiles this wavefront requests through the ring
  float best = 0.0f;
  for (int it = 0; it < cnt; ++it) {
    const int ahead = it + STAGES - 1;
    if (ahead < cnt)
      dma.issue(vg, first + (long long)ahead * WAVES, n, lane, ring + (ahead % STAGES) * T::kTileChunks);
    else if (CHAIN > 0 && ahead < total)
      dma.issue(next, next_first + (long long)(ahead - cnt) * CHAIN, n, lane, ring + (ahead % STAGES) * T::kTileChunks);
    const int younger = total - 1 - it < STAGES - 1 ? total - 1 - it : STAGES - 1;
    wait_tile<DT, D>(younger);
    // each lane sums the half row it holds (row lane % 32; rows past n repeat row n - 1), the two
    // halves are added across lanes
    u32x4 f[T::kSteps];
    frags.read(ring_addr + (it % STAGES) * T::kTileBytes, f);
    float s = 0.0f;
#pragma unroll
    for (int j = 0; j < T::kSteps; ++j) s = abs_sum16<DT>(f[j], s);
    s = add_halves(s);
    best = fmaxf(best, s);
    if (token_norm) {                                          // uniform: the rows' own norms, for the pooling step
      const long long row = (first + (long long)it * WAVES) * kTileKeys + (lane & 31);
      if (lane < 32 && row < n) row_norm[row] = s;
    }
  }
  return best;
}

// ------------------------------------------------------------------------------------------
// stats: per workgroup and per (head of the chunk, window row) the running maximum of the raw
// dot products and sum of exp2((dot - max) * c2) over the workgroup's keys, c2 = scale * log2 e.
// Row r may see keys 0 .. n - w + r only (each window row is normalised over the keys up to
// and including its own position).
// ------------------------------------------------------------------------------------------
//
// VN: the workgroup of a head's first chunk first sweeps the same span of the head's VALUE rows for their
// L1 norms (what vnorm_kernel does in a launch of its own, cut here like the statistics: vnorm_blocks ==
// blocks_x), through the same ring, and runs on into the keys without draining it.  One launch instead of
// two: one start-up and one tail for both streams.  Workgroup (0, 0) also clears what vnorm_kernel clears.
//
// NC: chunks of the group a workgroup handles, each by its own kWaves / NC wavefronts (SweepPlan::wg_chunks).
template <int DT, int D, int GT, int W, bool VN, int NC>
__global__ void __launch_bounds__((Shape<DT, D, W>::kThreads), (Shape<DT, D, W>::kMinWaves))
stats_kernel(const SweepArgs a) {
  using T = Tile<DT, D>;
  const Unit u = unit_of_block(a);
  const SweepSeq sq = a.s[u.z];
  const long long n = sq.n;
  const int w = a.w, G = a.G, n_chunks = a.n_chunks, tiles_per_block = sq.tiles_per_block;
  const RowMap rm = row_map(a);
  const float c2 = a.c2;
  const u32x4* __restrict__ q_win =
      static_cast<const u32x4*>(a.q_win) + (long long)(a.first_seq + u.z) * a.H * w * T::kCpr;
  const u32x4* __restrict__ k = static_cast<const u32x4*>(a.k) + (long long)a.H_kv * sq.tok * T::kCpr;
  float2* __restrict__ stat_part = reinterpret_cast<float2*>(a.ws + sq.ws_off + a.off_stat_part);
  constexpr int kWaves = Shape<DT, D, W>::kWaves;
  constexpr int kStages = Shape<DT, D, W>::kStages;
  __shared__ u32x4 s_tile[kWaves][kStages][T::kTileChunks];
  __shared__ float2 s_red[kWaves][kMaxChunkHeads * 32];   // [wave][head*32+row]

  const int lane = threadIdx.x & 63, wave = wave_index();
  constexpr int kPerChunk = kWaves / NC;                       // wavefronts of a chunk
  const int wave_chunk = wave / kPerChunk, wave_in_chunk = wave % kPerChunk;
  const int g = u.y / n_chunks, chunk = NC == 1 ? u.y % n_chunks : wave_chunk;
  const int head0 = NC > 2 && chunk * GT >= G ? G - 1 : chunk * GT;   // three chunks of four: the last one repeats a head, unused
  const int h0 = g * G + head0;
  const int nh = (G - head0) < GT ? (G - head0) : GT;
  const char* kg = reinterpret_cast<const char*>(k) + (long long)g * n * T::kRowBytes;

  TileDma<DT, D> dma;
  dma.init(lane);
  FragReader<DT, D> frags;
  frags.init(lane);

  const long long n_tiles = (n + kTileKeys - 1) / kTileKeys;
  const long long t_begin = (long long)u.x * tiles_per_block;
  long long t_end = t_begin + tiles_per_block;
  if (t_end > n_tiles) t_end = n_tiles;

  // this wavefront's key tiles: t_begin + its index in the chunk, + kPerChunk, ...; ring of kStages buffers,
  // kStages-1 tiles ahead.  Value tiles go round all wavefronts.
  const long long first = t_begin + wave_in_chunk;
  const int cnt = first < t_end ? (int)((t_end - first + kPerChunk - 1) / kPerChunk) : 0;
  u32x4* ring = s_tile[wave][0];
  const bool with_v = VN && (NC > 1 || chunk == 0);            // uniform
  const long long first_v = t_begin + wave;
  const int cnt_v = with_v && first_v < t_end ? (int)((t_end - first_v + kWaves - 1) / kWaves) : 0;
  const char* vg = nullptr;
  if constexpr (VN) {
    const u32x4* __restrict__ v = static_cast<const u32x4*>(a.v) + (long long)a.H_kv * sq.tok * T::kCpr;
    vg = reinterpret_cast<const char*>(v) + (long long)g * n * T::kRowBytes;
    if (u.x == 0 && u.y == 0) {
      uint32_t* __restrict__ counters = reinterpret_cast<uint32_t*>(a.ws + sq.ws_off + a.off_counter);
      const int n_counter_words = kCtlUnitA + a.H_kv * sq.blocks_x;
      for (int i = threadIdx.x; i < n_counter_words; i += Shape<DT, D, W>::kThreads) counters[i] = 0u;
      clear_selection_region(a, (int)u.z, Shape<DT, D, W>::kThreads);
    }
  }
  // VN: the query rows, once per workgroup, ahead of the first tiles: a chunk's heads into the last stage of its
  // wavefronts' rings, or, where it has fewer wavefronts than heads, into all stages (the first tiles then wait
  // until the rows are read).
  constexpr int kQSlots = GT <= kPerChunk ? 1 : GT / kPerChunk;    // heads a wavefront stages
  static_assert(kQSlots <= kStages, "one staging buffer per head");
  constexpr bool kQFirst = kQSlots > 1;
  auto q_buffer = [&](int t) { return s_tile[wave_chunk * kPerChunk + t / kQSlots][kStages - 1 - t % kQSlots]; };
  if constexpr (VN) {
#pragma unroll
    for (int i = 0; i < kQSlots; ++i) {
      const int t = wave_in_chunk * kQSlots + i;
      if (t < GT) request_q<DT, D, NC * GT>(dma, q_win, h0, nh, t, rm, lane, q_buffer(t));
    }
  }
  // with the value rows first, the ring holds both streams in turn: the wavefront's cnt_v value tiles, then
  // its cnt key tiles (a wavefront with few tiles already requests keys here)
  auto first_tiles = [&]() {
#pragma unroll
    for (int p = 0; p < kStages - 1; ++p) {
      if (p < cnt_v) dma.issue(vg, first_v + (long long)p * kWaves, n, lane, ring + p * T::kTileChunks);
      else if (p < cnt_v + cnt) dma.issue(kg, first + (long long)(p - cnt_v) * kPerChunk, n, lane, ring + p * T::kTileChunks);
    }
  };
  if constexpr (!(VN && kQFirst)) first_tiles();
  // VN: the value rows, which need no query rows, come first, so the wavefronts have drifted apart again by the
  // time the keys begin.  Every wavefront fetching its own copy of the query rows (eight times the traffic on lines
  // all workgroups want at once, and a wait for the first tiles as well) began the sweep 7.3 us after the
  // workgroup, staging them 3.5 us: 4115 tokens 14.6 -> 9.4 us for the launch, 32768 31.6 -> 29.4, 131072
  // 106 -> 102.
  // Otherwise every wavefront fetches its own copy, after its first tiles so that the two latencies
  // overlap.  (Staging was measured slower there: the wavefronts leave the barrier in step and the sweep loses
  // more than the set-up gains.)  Both are in before the loop: otherwise the compiler, which cannot count
  // the ring's loads across iterations, waits for everything in flight before each tile's products.
  u32x4 qf[GT][kQVec<DT, D>];
  bool q_parts = true;
  if constexpr (VN) {
    int young = 0;
    if constexpr (!kQFirst) {
#pragma unroll
      for (int p = 0; p < kStages - 1; ++p) young += p < cnt_v + cnt ? 1 : 0;
    }
    if (wave_in_chunk * kQSlots < GT) wait_tile<DT, D>(young);
    wave_barrier();
#pragma unroll
    for (int t = 0; t < GT; ++t) {
      u32x4 raw[T::kSteps];
      frags.read(lds_addr(q_buffer(t)), raw);
      q_parts &= make_q<DT, D>(raw, qf[t]);
    }
    wave_barrier();
    if constexpr (kQFirst) first_tiles();
  } else {
    q_parts = load_q<DT, D, GT>(q_win, h0, nh, rm, lane, qf);
    wait_vmcnt<0>();
  }
  q_parts = __ballot(!q_parts) == 0ull;
  float v_best = 0.0f;
  int slot0 = 0;
  if constexpr (VN) {
    if (with_v) {
      v_best = vnorm_tiles<DT, D, kWaves, kStages, kPerChunk>(
          dma, frags, vg, kg, n, first_v, cnt_v, first, cnt, ring, lane, a.token_norm != 0,
          a.scores + (long long)a.H_kv * sq.tok + (long long)g * n);
      slot0 = cnt_v % kStages;
    }
  }
  float m_run[GT], z_run[GT];
  stats_tiles<DT, D, GT, kPerChunk, kStages>(dma, frags, kg, n, rm, c2, first, cnt, ring, qf, q_parts, lane, m_run,
                                             z_run, slot0);
  if constexpr (VN) {
    __shared__ float s_vmax[kWaves];
    v_best = wave_max_f32(v_best);
    if (lane == 0) s_vmax[wave] = v_best;                      // read after the barrier of the merge below
    float2 mine;
    const bool owner = stats_merge_waves<GT, kWaves, NC>(m_run, z_run, c2, lane, wave, s_red, mine);
    if (owner) stat_part[((long long)(unsigned int)(u.y * sq.blocks_x + u.x)) * (NC * GT * 32) + threadIdx.x] = mine;
    if (with_v && threadIdx.x == 0) {
      float m = s_vmax[0];
#pragma unroll
      for (int i = 1; i < kWaves; ++i) m = fmaxf(m, s_vmax[i]);
      float* __restrict__ vnorm_part = reinterpret_cast<float*>(a.ws + sq.ws_off + a.off_vnorm_part);
      vnorm_part[(long long)g * sq.vnorm_blocks + u.x] = m;
    }
    if (with_v) clear_raw_scores(a, sq, g, t_begin, t_end, Shape<DT, D, W>::kThreads);
  } else {
    float2 mine;
    if (stats_merge_waves<GT, kWaves, NC>(m_run, z_run, c2, lane, wave, s_red, mine))
      stat_part[((long long)(unsigned int)(u.y * sq.blocks_x + u.x)) * (NC * GT * 32) + threadIdx.x] = mine;
  }
}

// ------------------------------------------------------------------------------------------
// scores: s_raw[g, i] = max over the heads h of group g of (1/w) sum_r softmax_r[h, i], i < n'.
// The normaliser of each (head, row) is merged from the stats partials by every workgroup, always
// in the same fixed order (deterministic) and with independent loads, or taken from a
// caller-supplied log-sum-exp.
// ------------------------------------------------------------------------------------------
//
// FUSED (all heads of the group in one workgroup, at most Shape::kFusedTiles tiles per workgroup): the
// workgroup keeps the raw scores of its key span in LDS, recomputes one tile on either side of
// the span (the pooling halo; 2 extra tiles per workgroup instead of a trip through HBM and
// another launch), and finishes the scores itself: max-pool, value factor, +inf for the window
// entries, and the layer statistic.  Otherwise the raw scores go to s_raw for poolstat_kernel.
constexpr int kPoolMaxHalf = 7;   // pooling kernels up to 15

struct PoolArgs {
  const float* vnorm_part;   // [H_kv][vnorm_blocks] value-norm partials
  int vnorm_blocks;
  int pool_half;
  int token_norm;            // scores[g][i] holds ||V[g, i]||_1 on entry: the value factor of entry i
  float* scores;             // [H_kv][n]
  float* vbar;               // [H_kv]
  float* layer_stat;         // [1]
  double2* ent_part;         // [workgroups]
  uint32_t* counters;
  const uint32_t* error_word; // persistent launch: non-zero once a wait for other workgroups gave up (statistic -> NaN); else null
  unsigned int* sel_hist0;    // first-digit histogram of the selection that will rank these scores, or null
  BudgetPlanArgs plan;        // budgets right after the statistic (e == nullptr: none)
  int plan_seq;               // the sequence's row in the plan's tables
};

// Histogram of the selection's first digit over the scores a workgroup has just written, for a selection
// workspace prepared alongside (lava_window_scores_primed): per-workgroup counts in `bins` (kSelDigit0Bins words
// of LDS, zeroed and published by a barrier before the first call), then one device-scope add per
// non-empty bin.  Runs of equal digits (pooling makes plateaus) are counted once per run by the caller.
__device__ __forceinline__ void digit0_count(unsigned int* bins, float score, unsigned int& run_digit,
                                             unsigned int& run_len) {
  const unsigned int digit = sel_digit0(score_key(score));
  if (digit != run_digit) {
    if (run_len != 0u) atomicAdd(&bins[run_digit], run_len);
    run_digit = digit;
    run_len = 0u;
  }
  ++run_len;
}
template <int THREADS>
__device__ __forceinline__ void digit0_flush(unsigned int* bins, unsigned int run_digit, unsigned int run_len,
                                             unsigned int* __restrict__ global_hist) {
  if (run_len != 0u) atomicAdd(&bins[run_digit], run_len);
  __syncthreads();
  for (int i = threadIdx.x; i < kSelDigit0Bins; i += THREADS) {
    const unsigned int c = bins[i];
    if (c) __hip_atomic_fetch_add(&global_hist[i], c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

// Exponent bias of every (head, row) of a scores workgroup, step 1: the head's statistics partials are cut into
// kMergeSlices runs of workgroups; "merger" (slice, row) merges its run in workgroup order into
// s_merge[slice][row] (always the same fixed order, independent loads: deterministic, no tickets).  In a workgroup
// with wavefronts to spare the mergers are those that do not fetch query rows.  DEVICE_SCOPE: the partials were
// written by other workgroups of the SAME launch (device-scope stores), so they are read with device-scope
// loads.  `part` points at partial 0 of the head's (chunk's) rows.  LDS is accessed by instruction here, so that
// tiles requested before stay in flight; the caller synchronises afterwards.
template <int GT, int WAVES>                                  // GT: heads of all chunks of the workgroup
struct Merge {
  static constexpr int kRows = GT * 32;
  static constexpr bool kSplit = WAVES >= 2 * GT;             // wavefronts GT .. merge, the others fetch query rows
  static constexpr int kThreads = (kSplit ? WAVES - GT : WAVES) * 64;
  static constexpr int kSlices = kThreads / kRows;
  static_assert(kSlices >= 1, "a merger per row");
};
template <int GT, int WAVES, bool DEVICE_SCOPE>
__device__ __forceinline__ void merge_partials(int merger, const float2* __restrict__ part, int stat_blocks, float c2,
                                               const float2* s_merge) {
  using M = Merge<GT, WAVES>;
  constexpr int kRows = M::kRows;
  if (merger < 0 || merger >= M::kSlices * kRows) return;
  const int row = merger % kRows, slice = merger / kRows;
  float m = -INFINITY, z = 0.0f;
  const int per = (stat_blocks + M::kSlices - 1) / M::kSlices;
  const int b_begin = slice * per, b_end = (b_begin + per < stat_blocks) ? b_begin + per : stat_blocks;
  const float2* p = part + row;
  for (int b0 = b_begin; b0 < b_end; b0 += 16) {
    float2 x[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      if (b0 + u < b_end)
        x[u] = DEVICE_SCOPE ? ld_dev_f2(&p[(long long)(b0 + u) * kRows]) : p[(long long)(b0 + u) * kRows];
      else
        x[u] = make_float2(-INFINITY, 0.0f);
    }
    merge_stats<16>(x, c2, m, z);
  }
  lds_write64(lds_addr(s_merge) + (unsigned int)(slice * kRows + row) * 8u, make_float2(m, z));
}

// Step 2: the slices are merged in slice order; bias = log2(row normaliser * w) in the exp2 domain,
// +inf for padding rows (their exponentials vanish).  Thread t < kRows does row t.
template <int GT, int WAVES>
__device__ __forceinline__ void write_bias(const float2* s_merge, int nh, int h0, const RowMap& rm, float c2, const float* s_bias) {
  using M = Merge<GT, WAVES>;
  if (threadIdx.x >= M::kRows) return;
  const int t = threadIdx.x >> 5;
  float m = -INFINITY, z = 0.0f;
#pragma unroll
  for (int sl = 0; sl < M::kSlices; ++sl) {
    const float2 x = lds_read64(lds_addr(s_merge) + (unsigned int)(sl * M::kRows + (int)threadIdx.x) * 8u);
    merge_stat(m, z, x.x, x.y, c2);
  }
  const bool real = t < nh && row_at<GT>(rm, h0 + t, (int)(threadIdx.x & 31)).real;
  const float bias = real ? m * c2 + log2f(z) + log2f((float)rm.w) : INFINITY;
  lds_write32(lds_addr(s_bias) + threadIdx.x * 4u, bias);
}
// ... or the bias of the caller's log-sum-exp, by merger t < kRows
template <int GT>
__device__ __forceinline__ void bias_of_lse(int merger, const float* __restrict__ lse, int nh, int h0, const RowMap& rm,
                                            const float* s_bias) {
  if (merger < 0 || merger >= GT * 32) return;
  const int t = merger >> 5;
  const RowAt at = row_at<GT>(rm, h0 + t, merger & 31);
  float bias = INFINITY;
  if (t < nh && at.real) bias = lse[(long long)at.head * rm.w + at.row] * kLog2e + log2f((float)rm.w);
  lds_write32(lds_addr(s_bias) + (unsigned int)merger * 4u, bias);
}

// Raw score of this lane's key (lane % 32 of the tile whose fragments are in kf): maximum over the chunk's heads of the
// window mean of the attention.  bias_addr: LDS address of the chunk's biases, + 16 for the upper lane half (rows held by
// a lane in result register v: 8 * (v / 4) + 4 * half + v % 4 -> four float4 per head).
template <int DT, int D, int GT>
__device__ __forceinline__ float score_tile(const u32x4 (&kf)[Tile<DT, D>::kSteps], float c2, unsigned int bias_addr,
                                            const u32x4 (&qf)[GT][kQVec<DT, D>], bool q_parts, const RowMap& rm) {
  float best = 0.0f, pair = 0.0f;
  f32x16 all[DT == LAVA_F32 ? GT : 1];
  if constexpr (DT == LAVA_F32) dot_tiles<D, GT, false>(kf, qf, q_parts, all);
  auto head_dots = [&](int t) -> f32x16 {
    if constexpr (DT == LAVA_F32) return all[t];
    else return dot_tile<D, false>(kf, qf[t]);
  };
  f32x16 acc = head_dots(0);
#pragma unroll
  for (int t = 0; t < GT; ++t) {
    f32x16 nxt = acc;
    if (t + 1 < GT) nxt = head_dots(t + 1);
    u32x4 bb[4];                       // biases of rows 8*jj + 4*half + 0..3 of block t
    lds_read128x4_strided<32>(bias_addr + t * 128, bb[0], bb[1], bb[2], bb[3]);
    auto share = [&](float sum, int jj) {   // + the exponentials of four rows
      sum += fast_exp2(fmaf(acc[4 * jj + 0], c2, -__uint_as_float(bb[jj].x)));
      sum += fast_exp2(fmaf(acc[4 * jj + 1], c2, -__uint_as_float(bb[jj].y)));
      sum += fast_exp2(fmaf(acc[4 * jj + 2], c2, -__uint_as_float(bb[jj].z)));
      sum += fast_exp2(fmaf(acc[4 * jj + 3], c2, -__uint_as_float(bb[jj].w)));
      return sum;
    };
    if constexpr (GT == 1) {             // the one case in which heads share a block (sweep_rows_per_head)
      if (rm.rph == 8) {                 // uniform
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) best = fmaxf(best, add_halves(share(0.0f, jj)));
        break;
      }
      if (rm.rph == 16) {
        best = fmaxf(best, add_halves(share(share(0.0f, 0), 1)));   // a NaN does not count, so the score stays a number
        best = fmaxf(best, add_halves(share(share(0.0f, 2), 3)));
        break;
      }
    }
    float ps = 0.0f;
#pragma unroll
    for (int jj = 0; jj < 4; ++jj) ps = share(ps, jj);
    ps = add_halves(ps);
    if (rm.bph == 2) {                   // uniform: a head's window mean is the sum over its two row blocks
      if (t & 1) best = fmaxf(best, pair + ps);
      else pair = ps;
    } else {
      best = fmaxf(best, ps);
    }
    acc = nxt;
  }
  return best;
}

// This lane's raw score into a tile's place in the span of raw scores; JOIN: as a maximum.  The lane's slot is formed
// from the lane counter instead of living in a register across the loop, which has none to spare.
template <bool JOIN>
__device__ __forceinline__ void span_put(unsigned int tile_at, float score) {
  unsigned int l;
  asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(l));
  if (l < 32u) {
    if constexpr (JOIN) lds_max32(tile_at + l * 4u, score);
    else lds_write32(tile_at + l * 4u, score);
  }
}

// The score sweep of one wavefront over the jobs of its workgroup: the workgroup's own tiles
// t_begin .. t_end - 1, then (FUSED) the pooling halo, i.e. the tile before and the tile after the
// span.  fifo[] holds the jobs this wavefront has already requested into its ring (the first
// STAGES - 1 are fixed); the rest are taken from the shared counter *next_job as wavefronts become
// free, because the wavefronts of a workgroup do not run at the same speed.  Which wavefront
// computes a tile does not change its result, so the scores stay deterministic.
// FUSED: raw scores go to s_span (position p of the prefix at s_span[p - (t_begin - 1) * 32]; SHARED_SPAN: as a
// maximum, joined with what the wavefronts of the group's other chunk find);
// otherwise to raw_head[position] (atomic maximum when the group is split over workgroups).
template <int DT, int D, int GT, int WAVES, int STAGES, bool FUSED, bool SHARED_SPAN>
__device__ __forceinline__ void scores_tiles(const TileDma<DT, D>& dma, const FragReader<DT, D>& frags,
                                             const char* __restrict__ kg, long long n, long long n_prefix, float c2,
                                             long long t_begin, long long t_end, int n_own, bool halo_left,
                                             bool halo_right, int n_jobs, int (&fifo)[STAGES], u32x4* ring,
                                             unsigned int* next_job, const float* s_bias, float* s_span,
                                             const u32x4 (&qf)[GT][kQVec<DT, D>], bool q_parts, int lane,
                                             float* __restrict__ raw_head, int n_chunks, const RowMap& rm) {
  using T = Tile<DT, D>;
  auto job_tile = [&](int j) -> long long {
    if (j < n_own) return t_begin + j;
    return (j == n_own && halo_left) ? t_begin - 1 : t_end;
  };
  (void)halo_right;
  const int half = lane >> 5;
  const unsigned int ring_addr = lds_addr(ring);
  const unsigned int next_job_addr = lds_addr(next_job);
  const unsigned int bias_addr = lds_addr(s_bias) + half * 16;
  const unsigned int span_base = lds_addr(s_span);

  // The result of a tile is stored one iteration later, right after the next tile's arrival wait:
  // the store then has a whole iteration to complete before a wait counts it among the older
  // operations, instead of stalling every iteration on its acknowledgement.
  float pend = 0.0f;
  int pend_key = -1;                 // n < 2^31
  auto store_result = [&](int key, float value) {
    if (half == 0 && key >= 0 && key < n_prefix) {
      float* dst = raw_head + key;
      if (n_chunks == 1) {
        *dst = value;
      } else {   // heads of the group are split over workgroups: non-negative floats order as integers
        atomicMax(reinterpret_cast<unsigned int*>(dst), __float_as_uint(value));
      }
    }
  };
  bool more = true;                                             // the counter has not run out yet
  for (int it = 0; fifo[0] >= 0; ++it) {
    const long long tile = job_tile(fifo[0]);
    if (more) {
      unsigned int j = 0;
      if (lane == 0) j = lds_fetch_inc(next_job_addr);
      j = __builtin_amdgcn_readfirstlane(j);
      more = j < (unsigned int)n_jobs;
      if (more) {
        fifo[STAGES - 1] = (int)j;
        dma.issue(kg, job_tile((int)j), n, lane, ring + ((it + STAGES - 1) % STAGES) * T::kTileChunks);
      }
    }
    int younger = 0;
#pragma unroll
    for (int p = 1; p < STAGES; ++p) younger += fifo[p] >= 0 ? 1 : 0;
    wait_tile<DT, D>(younger);
#pragma unroll
    for (int p = 0; p + 1 < STAGES; ++p) fifo[p] = fifo[p + 1];
    fifo[STAGES - 1] = -1;
    if constexpr (!FUSED) store_result(pend_key, pend);
    u32x4 kf[T::kSteps];
    frags.read(ring_addr + (it % STAGES) * T::kTileBytes, kf);
    const float best = score_tile<DT, D, GT>(kf, c2, bias_addr, qf, q_parts, rm);
    if constexpr (FUSED) {
      span_put<SHARED_SPAN>(span_base + (unsigned int)(tile - t_begin + 1) * (kTileKeys * 4), best);
    } else {
      pend = best;
      pend_key = (int)(tile * kTileKeys) + (lane & 31);
    }
  }
  if constexpr (!FUSED) store_result(pend_key, pend);
}

// Finishes the scores of a workgroup's span from the raw scores in s_span (FUSED): Vbar of the head
// (vb: this thread's share of the head's value-norm partials), max-pool over the prefix, the value
// factor, +inf for the window entries, and the workgroup's share of the layer statistic; the last
// workgroup of the sequence to arrive (block_id of n_blocks) forms e.  Contains workgroup barriers.
template <int THREADS>
__device__ __forceinline__ void scores_finish(const PoolArgs& pa, float vb, int g, long long n, long long n_prefix, int w,
                                              long long t_begin, long long t_end, long long n_tiles,
                                              const float* s_span, float* s_vb, double* s_s, double* s_t,
                                              unsigned int* s_last, unsigned int n_blocks, unsigned int block_id,
                                              int n_heads, bool writes_vbar, int wave, unsigned int* bins) {
  constexpr int kWaves = THREADS / 64;
  // `bins`: kSelDigit0Bins words of LDS that only wavefront 0 has used since the workgroup's last barrier (the
  // start of its own tile ring, which it is done with)
  const bool count_digits = pa.sel_hist0 != nullptr;
  const PlanInputs plan_in = plan_prefetch(pa.plan, pa.plan_seq);
  if (count_digits && wave == 0)
    for (int i = threadIdx.x; i < kSelDigit0Bins; i += 64) bins[i] = 0u;
  unsigned int run_digit = 0u, run_len = 0u;
  vb = wave_max_f32(vb);
  if ((threadIdx.x & 63) == 0) s_vb[wave] = vb;
  lds_reads_done();                      // this wavefront's span entries are written
  __syncthreads();                       // s_span complete, s_vb visible
  vb = s_vb[0];
#pragma unroll
  for (int i = 1; i < kWaves; ++i) vb = fmaxf(vb, s_vb[i]);
  if (writes_vbar && threadIdx.x == 0) pa.vbar[g] = vb;

  const long long p_begin = t_begin * kTileKeys;
  long long p_end = t_end * kTileKeys;
  if (p_end > n_prefix) p_end = n_prefix;
  const long long span0 = (t_begin - 1) * kTileKeys;      // position held by s_span[0]
  // kPer consecutive positions per thread: kPer + 16 raw scores (positions base-8 .. base+kPer+7) cover every tap
  // of a pooling window of up to 15; positions outside the prefix do not take part in the maximum (the
  // window is clipped, not padded).  Eight where the span has work for all threads (six 128-bit reads), two
  // where it is short: a thread's logarithms are a serial chain.
  double acc_s = 0.0, acc_t = 0.0;
  static_assert(kPoolMaxHalf <= 8, "taps must stay inside the values read");
  const float* out_head = pa.scores + (long long)g * n;
  auto pool = [&](auto per) {
    constexpr int kPer = decltype(per)::value;
    constexpr int kVec = kPer < 4 ? kPer : 4;
    typedef float vec __attribute__((ext_vector_type(kVec)));
    for (long long base = p_begin + (long long)threadIdx.x * kPer; base < p_end; base += (long long)THREADS * kPer) {
      float raw[kPer + 16];
      const vec* src = reinterpret_cast<const vec*>(&s_span[(int)(base - 8 - span0)]);
#pragma unroll
      for (int i = 0; i < (kPer + 16) / kVec; ++i) {
        const vec x = src[i];
#pragma unroll
        for (int e = 0; e < kVec; ++e) raw[kVec * i + e] = x[e];
      }
#pragma unroll
      for (int i = 0; i < kPer + 16; ++i) {
        const long long pos = base - 8 + i;
        if (pos < 0 || pos >= n_prefix) raw[i] = -INFINITY;
      }
      float sc[kPer];
#pragma unroll
      for (int j = 0; j < kPer; ++j) sc[j] = raw[8 + j];
#pragma unroll
      for (int dd = 1; dd <= kPoolMaxHalf; ++dd) {
        if (dd <= pa.pool_half) {                              // uniform
#pragma unroll
          for (int j = 0; j < kPer; ++j) sc[j] = fmaxf(sc[j], fmaxf(raw[8 + j - dd], raw[8 + j + dd]));
        }
      }
      float fac[kPer];
#pragma unroll
      for (int j = 0; j < kPer; ++j) fac[j] = vb;
      if (pa.token_norm) {                                     // uniform
#pragma unroll
        for (int j = 0; j < kPer; ++j)
          if (base + j < p_end) fac[j] = out_head[base + j];
      }
#pragma unroll
      for (int j = 0; j < kPer; ++j) {
        sc[j] *= fac[j];
        if (base + j < p_end) {
          acc_s += (double)sc[j];
          if (sc[j] > 0.0f) acc_t += (double)sc[j] * (double)logf(sc[j]);
          if (count_digits) digit0_count(bins, sc[j], run_digit, run_len);
        }
      }
      if (base + kPer <= p_end && (reinterpret_cast<uintptr_t>(out_head + base) & (4 * kVec - 1)) == 0) {
        vec* dst = reinterpret_cast<vec*>(const_cast<float*>(out_head) + base);
#pragma unroll
        for (int i = 0; i < kPer / kVec; ++i) {
          vec x;
#pragma unroll
          for (int e = 0; e < kVec; ++e) x[e] = sc[kVec * i + e];
          dst[i] = x;
        }
      } else {
#pragma unroll
        for (int j = 0; j < kPer; ++j)
          if (base + j < p_end) pa.scores[(long long)g * n + base + j] = sc[j];
      }
    }
  };
  if (p_end - p_begin <= 2 * THREADS) pool(std::integral_constant<int, 2>{});   // uniform
  else pool(std::integral_constant<int, 8>{});
  // the workgroup that owns the head's last prefix tile also writes the window entries
  if (t_begin < t_end && t_end == n_tiles && threadIdx.x < (unsigned)w) {
    pa.scores[(long long)g * n + n_prefix + threadIdx.x] = INFINITY;
    if (count_digits) digit0_count(bins, INFINITY, run_digit, run_len);
  }
  if (count_digits) digit0_flush<THREADS>(bins, run_digit, run_len, pa.sel_hist0);
  const bool last = entropy_finish<THREADS>(acc_s, acc_t, pa.ent_part, pa.counters, n_blocks, block_id,
                                            (double)n_heads * (double)n_prefix, pa.layer_stat, s_s, s_t, s_last,
                                            pa.error_word);
  if (last && pa.plan.e != nullptr) {                        // uniform
    __syncthreads();                                         // s_t[0]; every wavefront is done with `bins`
    // scratch: what is left of wavefront 0's own tile ring behind the bins
    static_assert(kSelDigit0Bins * 4 + sizeof(BudgetScratchT<kMaxPlannedLayers>) <= 16 * 1024, "wavefront 0's ring");
    plan_budgets(pa.plan, plan_in, pa.plan_seq, (float)s_t[0], bins + kSelDigit0Bins);
  }
}

template <int DT, int D, int GT, bool FUSED, int W, int NC>
__global__ void __launch_bounds__((Shape<DT, D, W>::kThreads), (Shape<DT, D, W>::kMinWaves))
scores_kernel(const SweepArgs a) {
  using T = Tile<DT, D>;
  const Unit u = unit_of_block(a);
  const SweepSeq sq = a.s[u.z];
  const int seq = a.first_seq + (int)u.z;
  const long long n = sq.n;
  const int w = a.w, G = a.G, n_chunks = a.n_chunks, tiles_per_block = sq.tiles_per_block;
  const RowMap rm = row_map(a);
  const int stat_blocks = sq.blocks_x;
  const float c2 = a.c2;
  const u32x4* __restrict__ q_win = static_cast<const u32x4*>(a.q_win) + (long long)seq * a.H * w * T::kCpr;
  const u32x4* __restrict__ k = static_cast<const u32x4*>(a.k) + (long long)a.H_kv * sq.tok * T::kCpr;
  char* region = a.ws + sq.ws_off;
  const float2* __restrict__ stat_part = reinterpret_cast<const float2*>(region + a.off_stat_part);
  const float* __restrict__ lse = a.lse ? a.lse + (long long)seq * a.H * w : nullptr;
  float* __restrict__ s_raw = reinterpret_cast<float*>(region + a.off_sraw);
  PoolArgs pa;
  pa.vnorm_part = reinterpret_cast<const float*>(region + a.off_vnorm_part);
  pa.vnorm_blocks = sq.vnorm_blocks;
  pa.pool_half = a.pool_half;
  pa.scores = a.scores + (long long)a.H_kv * sq.tok;
  pa.vbar = a.vbar + (long long)seq * a.H_kv;
  pa.token_norm = a.token_norm;
  pa.layer_stat = a.layer_stat + seq;
  pa.ent_part = reinterpret_cast<double2*>(region + a.off_ent_part);
  pa.counters = reinterpret_cast<uint32_t*>(region + a.off_counter);
  pa.error_word = nullptr;
  pa.sel_hist0 = a.sel_ws ? reinterpret_cast<unsigned int*>(a.sel_ws + (size_t)seq * a.sel_stride + a.sel_off_hist) : nullptr;
  pa.plan = a.plan;
  pa.plan_seq = seq;
  constexpr int kWaves = Shape<DT, D, W>::kWaves;
  constexpr int kStages = Shape<DT, D, W>::kStages;
  __shared__ u32x4 s_tile[kWaves][kStages][T::kTileChunks];
  __shared__ __attribute__((aligned(16))) float s_bias[NC * GT * 32];
  __shared__ __attribute__((aligned(16))) float s_span[FUSED ? (Shape<DT, D, W>::kFusedTiles + 2) * kTileKeys : 4];   // raw scores of the span + halo tiles

  const int lane = threadIdx.x & 63, wave = wave_index();
  static_assert(NC == 1 || FUSED, "several chunks in a workgroup finish the scores there");
  constexpr int kPerChunk = kWaves / NC;                       // wavefronts of a chunk
  const int wave_chunk = wave / kPerChunk, wave_in_chunk = wave % kPerChunk;
  const int g = u.y / n_chunks, chunk = NC == 1 ? u.y % n_chunks : wave_chunk;
  const int head0 = NC > 2 && chunk * GT >= G ? G - 1 : chunk * GT;   // three chunks of four: the last one repeats a head, unused
  const int h0 = g * G + head0;
  const int nh = (G - head0) < GT ? (G - head0) : GT;
  const int wg_h0 = NC == 1 ? h0 : g * G, wg_nh = NC == 1 ? nh : G;   // heads of the workgroup
  const char* kg = reinterpret_cast<const char*>(k) + (long long)g * n * T::kRowBytes;
  const long long n_prefix = n - w;

  float vb = 0.0f;   // this thread's share of the head's value-norm partials (reduced after the sweep)
  if constexpr (FUSED) {
    for (int i = threadIdx.x; i < pa.vnorm_blocks; i += Shape<DT, D, W>::kThreads)
      vb = fmaxf(vb, pa.vnorm_part[(long long)g * pa.vnorm_blocks + i]);
  }

  constexpr int kThreads = Shape<DT, D, W>::kThreads;
  using M = Merge<NC * GT, kWaves>;
  __shared__ float2 s_merge[M::kSlices * M::kRows];

  __shared__ unsigned int s_next_job[NC];
  if (threadIdx.x < NC) s_next_job[threadIdx.x] = kPerChunk * (kStages - 1);   // published by the barriers below
  TileDma<DT, D> dma;
  dma.init(lane);
  FragReader<DT, D> frags;
  frags.init(lane);
  const long long n_tiles = (n_prefix + kTileKeys - 1) / kTileKeys;
  const long long t_begin = (long long)u.x * tiles_per_block;
  long long t_end = t_begin + tiles_per_block;
  if (t_end > n_tiles) t_end = n_tiles;
  // Jobs of the workgroup: its own tiles, then (FUSED) the pooling halo, i.e. the tile before and the
  // tile after the span.  The first kStages - 1 jobs of every wavefront are fixed; the rest are taken
  // from a shared counter as wavefronts become free, because the wavefronts of a workgroup do not
  // run at the same speed (two share each SIMD and the older one wins the arbitration).  Which
  // wavefront computes a tile does not change its result, so the scores stay deterministic.  With two chunks
  // the workgroup has each job twice, once for the wavefronts of either chunk.
  const int n_own = t_begin < t_end ? (int)(t_end - t_begin) : 0;
  const bool halo_left = FUSED && n_own > 0 && t_begin > 0;
  const bool halo_right = FUSED && n_own > 0 && t_end < n_tiles;
  const int n_jobs = n_own + (halo_left ? 1 : 0) + (halo_right ? 1 : 0);
  auto job_tile = [&](int j) -> long long {
    if (j < n_own) return t_begin + j;
    return (j == n_own && halo_left) ? t_begin - 1 : t_end;
  };
  int fifo[kStages];                                            // jobs requested and not yet computed; -1: none
#pragma unroll
  for (int p = 0; p < kStages; ++p) {
    const int j = wave_in_chunk + p * kPerChunk;
    fifo[p] = (p < kStages - 1 && j < n_jobs) ? j : -1;
  }
  u32x4* ring = s_tile[wave][0];
  if constexpr (NC > 1)                                         // published by the barriers below
    for (int i = threadIdx.x; i < (n_own + 2) * kTileKeys; i += kThreads) lds_write32(lds_addr(s_span) + i * 4u, 0.0f);
  // Set-up: the first wavefronts request the query rows into the last stage of their rings (idle until the loop
  // starts) while the others merge the normalisers of every (head, row), from the statistics partials or the
  // caller's log-sum-exp; then everybody requests first tiles.  Loads return in order and the compiler cannot
  // count the conditional ones, so what is waited for goes out ahead of the tiles: with the tiles first and
  // the query rows copied through registers the loop began 7.2 us after the workgroup, of which 4.5 were the
  // first tiles' way (131072 tokens), and the device idled until the second ones arrived.
  // (Where a chunk has fewer wavefronts than heads, the query rows take every stage and the first tiles wait.)
  constexpr int kQSlots = GT <= kPerChunk ? 1 : GT / kPerChunk;    // heads a wavefront stages
  static_assert(kQSlots <= kStages, "one staging buffer per head");
  constexpr bool kQFirst = kQSlots > 1;
  auto q_buffer = [&](int t) { return s_tile[wave_chunk * kPerChunk + t / kQSlots][kStages - 1 - t % kQSlots]; };
  const auto request_rows = [&]() {
#pragma unroll
    for (int i = 0; i < kQSlots; ++i) {
      const int t = wave_in_chunk * kQSlots + i;
      if (t < GT) request_q<DT, D, NC * GT>(dma, q_win, h0, nh, t, rm, lane, q_buffer(t));
    }
    asm volatile("" ::: "memory");
  };
  if constexpr (!M::kSplit) request_rows();                     // ahead of the partials, whose wait covers both
  const int merger = M::kSplit ? (int)threadIdx.x - NC * GT * 64 : (int)threadIdx.x;
  if (lse != nullptr)
    bias_of_lse<NC * GT>(merger, lse, wg_nh, wg_h0, rm, s_bias);
  else
    merge_partials<NC * GT, kWaves, false>(merger, stat_part + (long long)u.y * stat_blocks * M::kRows, stat_blocks, c2, s_merge);
  asm volatile("" ::: "memory");
  if constexpr (M::kSplit) request_rows();
  int young = 0;
  auto first_tiles = [&]() {
#pragma unroll
    for (int p = 0; p < kStages - 1; ++p)
      if (fifo[p] >= 0) {
        dma.issue(kg, job_tile(fifo[p]), n, lane, ring + p * T::kTileChunks);
        ++young;
      }
  };
  if constexpr (!kQFirst) first_tiles();
  if (wave_in_chunk * kQSlots < GT) wait_tile<DT, D>(young);
  wave_barrier();
  if (lse == nullptr) write_bias<NC * GT, kWaves>(s_merge, wg_nh, wg_h0, rm, c2, s_bias);
  u32x4 qf[GT][kQVec<DT, D>];
  bool q_parts = true;
#pragma unroll
  for (int t = 0; t < GT; ++t) {
    u32x4 raw[T::kSteps];
    frags.read(lds_addr(q_buffer(t)), raw);
    q_parts &= make_q<DT, D>(raw, qf[t]);
  }
  q_parts = __ballot(!q_parts) == 0ull;
  wave_barrier();
  if constexpr (kQFirst) first_tiles();

  scores_tiles<DT, D, GT, kPerChunk, kStages, FUSED, (NC > 1)>(
      dma, frags, kg, n, n_prefix, c2, t_begin, t_end, n_own, halo_left, halo_right, n_jobs, fifo, ring,
      &s_next_job[NC == 1 ? 0 : wave_chunk], s_bias + (NC == 1 ? 0 : wave_chunk * GT * 32), s_span, qf, q_parts, lane,
      s_raw + (long long)g * n_prefix, n_chunks, rm);
  if constexpr (FUSED) {
    __shared__ float s_vb[kWaves];
    __shared__ double s_s[kWaves], s_t[kWaves];
    __shared__ unsigned int s_last;
    scores_finish<kThreads>(pa, vb, g, n, n_prefix, w, t_begin, t_end, n_tiles, s_span, s_vb, s_s, s_t, &s_last,
                            (unsigned int)(sq.blocks_x * a.H_kv), (unsigned int)(u.y * sq.blocks_x + u.x), a.H_kv,
                            u.x == 0, wave, reinterpret_cast<unsigned int*>(&s_tile[0][0][0]));
  }
}

// ------------------------------------------------------------------------------------------
// sweep: statistics and scores of a launch's sequences in ONE persistent launch.
//
// Work units are (sequence, KV head, span of keys): the same spans the two separate kernels give
// their workgroups.  Workgroup b of a grid of `grid` workgroups owns units b, b + grid, ... : it
// first runs their statistics passes, then their score passes.  A score unit needs the statistics
// of all spans of its head: it waits for the head's completion count.  So that this wait cannot
// depend on the whole grid being resident, every statistics unit carries a claim word: its owner
// claims it (a compare-and-swap on a word nobody else touches, in flight while the unit's first
// tiles are requested), and a workgroup whose wait lasts long looks for unclaimed statistics units
// of the head it waits for and runs them itself (it already holds that head's query rows).  A
// claimed unit is being run by a resident workgroup that waits for nothing, so every wait ends.
// (The waits are bounded all the same; one that gives up sets an error word and the layer
// statistic becomes NaN.)
// What the single launch saves over two: the query rows are fetched once, the second pass of a
// head starts as soon as that head's statistics are complete instead of after the slowest
// workgroup of the whole device, its first tiles are requested before the statistics are even
// published, and there is no second launch.  Results are bit-identical to the separate kernels:
// the same tiles are combined in the same order.
// ------------------------------------------------------------------------------------------
template <int DT, int D, int GT, int W>
struct SweepSmem {
  using T = Tile<DT, D>;
  using S = Shape<DT, D, W>;
  u32x4 tile[S::kWaves][S::kStages][T::kTileChunks];
  __attribute__((aligned(16))) float bias[GT * 32];
  union {
    float2 red[S::kWaves][kMaxChunkHeads * 32];            // statistics units: per-wavefront results
    struct {
      float2 merge[Merge<GT, S::kWaves>::kSlices * GT * 32];   // score units: slices of the partial merge
      __attribute__((aligned(16))) float span[(S::kFusedTiles + 2) * kTileKeys];   // raw scores of the span + halo
    } sc;
  };
  float vb[S::kWaves];
  double ss[S::kWaves], st[S::kWaves];
  unsigned int last, next_job;
  int claim[4];                                             // words handed from thread 0 to the workgroup
};

__device__ __forceinline__ void lds_write128(unsigned int a, const u32x4& x) {
  asm volatile("ds_write_b128 %0, %1" : : "v"(a), "v"(x) : "memory");
}

template <int DT, int D, int GT, int W>
__global__ void __launch_bounds__((Shape<DT, D, W>::kThreads), (Shape<DT, D, W>::kMinWaves))
sweep_kernel(const SweepArgs a) {
  using T = Tile<DT, D>;
  using S = Shape<DT, D, W>;
  constexpr int kWaves = S::kWaves, kStages = S::kStages, kThreads = S::kThreads, kRows = GT * 32;
  static_assert(kWaves >= GT, "one staging buffer per head");
  __shared__ SweepSmem<DT, D, GT, W> sm;
  const int lane = threadIdx.x & 63, wave = wave_index();
  const int w = a.w, G = a.G, H_kv = a.H_kv;
  const RowMap rm = row_map(a);
  const float c2 = a.c2;
  uint32_t* __restrict__ ctl0 = reinterpret_cast<uint32_t*>(a.ws + a.s[0].ws_off + a.off_counter);
  TileDma<DT, D> dma;
  dma.init(lane);
  FragReader<DT, D> frags;
  frags.init(lane);
  u32x4* ring = sm.tile[wave][0];

  // Query rows of (sequence si, head g), once per workgroup and unit.  The w rows of a head are one
  // contiguous run of q_win, i.e. a key tile of w rows: wavefront t requests head t's rows straight into
  // its idle last ring stage with the same direct-to-LDS loads (rows beyond the window repeat row w - 1,
  // heads beyond the group repeat its last head: their results are never used), AHEAD of the unit's first
  // key tiles, so that q_commit only waits for the older loads and the tiles stay in flight.
  // (Keeping the rows in registers from one unit to the next costs more registers than the two
  // passes leave.)  The workgroup is past a barrier since it last used those stages.
  auto q_request = [&](int si, int g) {
    if (wave < GT) {
      const int nh = G < GT ? G : GT;
      const int h = g * G + (wave < nh ? wave : nh - 1);
      const char* rows = static_cast<const char*>(a.q_win) +
                         ((long long)(a.first_seq + si) * a.H + h) * w * (long long)T::kRowBytes;
      dma.issue_clamped(rows, 0, w, lane, ring + (kStages - 1) * T::kTileChunks);
    }
  };
  // `younger`: key tiles this wavefront has requested since q_request
  auto q_commit = [&](u32x4 (&qf)[GT][kQVec<DT, D>], int younger) -> bool {
    if (wave < GT) wait_tile<DT, D>(younger);
    __syncthreads();
    bool parts = true;
#pragma unroll
    for (int t = 0; t < GT; ++t) {
      u32x4 raw[T::kSteps];
      frags.read(lds_addr(&sm.tile[t][kStages - 1][0]), raw);
      parts &= make_q<DT, D>(raw, qf[t]);
    }
    __syncthreads();
    return __ballot(!parts) == 0ull;
  };
  auto seq_of_unit = [&](int u) {
    int si = 0;
    while (si + 1 < a.n_seq && u >= a.s[si + 1].unit_base) ++si;
    return si;
  };

  // The workgroup's own units: u_a walks its statistics units, then u_b its score units.  A score unit
  // whose wait for its head's statistics lasts may hand a statistics unit of that head to the top of
  // the loop (help_bx >= 0) and is set up again afterwards; there is one copy of each pass's code.
  int u_a = (int)blockIdx.x, u_b = (int)blockIdx.x;
  int help_si = 0, help_g = 0, help_bx = -1;
  for (;;) {
    // ------------------------------------------------------------ a statistics unit, if there is one to run
    int si = 0, g = 0, bx = -1;
    if (help_bx >= 0) {
      si = help_si; g = help_g; bx = help_bx;
      help_bx = -1;
    } else if (u_a < a.n_units) {
      const int u = u_a;
      u_a += (int)gridDim.x;
      // testing aid: every orphan_mod-th unit is left alone by its owner, as if the owner were not resident;
      // somebody waiting for the unit's head has to run it (the helping path below)
      if (a.orphan_mod != 0 && (u % a.orphan_mod) == 0) continue;
      si = seq_of_unit(u);
      const int rel = u - a.s[si].unit_base;
      g = rel / a.s[si].blocks_x;
      bx = rel % a.s[si].blocks_x;
    }
    if (bx >= 0) {
      const SweepSeq sq = a.s[si];
      const long long n = sq.n;
      const char* kg = static_cast<const char*>(a.k) + ((long long)H_kv * sq.tok + (long long)g * n) * T::kRowBytes;
      char* region = a.ws + sq.ws_off;
      float2* __restrict__ stat_part = reinterpret_cast<float2*>(region + a.off_stat_part);
      uint32_t* __restrict__ ctl = reinterpret_cast<uint32_t*>(region + a.off_counter);
      const long long n_tiles = (n + kTileKeys - 1) / kTileKeys;
      const long long t_begin = (long long)bx * sq.tiles_per_block;
      long long t_end = t_begin + sq.tiles_per_block;
      if (t_end > n_tiles) t_end = n_tiles;
      const long long first = t_begin + wave;
      const int cnt = first < t_end ? (int)((t_end - first + kWaves - 1) / kWaves) : 0;
      // Exactly the statistics kernel's pass: every wavefront fetches its own copy of the query rows after
      // its first tiles and enters the loop when both are in, without a workgroup barrier in front of
      // the loop (one there costs the pass a fifth of its speed, measured).
#pragma unroll
      for (int p = 0; p < kStages - 1; ++p)
        if (p < cnt) dma.issue(kg, first + (long long)p * kWaves, n, lane, ring + p * T::kTileChunks);
      u32x4 qf[GT][kQVec<DT, D>];
      bool q_parts = load_q<DT, D, GT>(static_cast<const u32x4*>(a.q_win) + (long long)(a.first_seq + si) * a.H * w * T::kCpr, g * G,
                                        G < GT ? G : GT, rm, lane, qf);
      wait_vmcnt<0>();
      q_parts = __ballot(!q_parts) == 0ull;
      float m_run[GT], z_run[GT];
      stats_tiles<DT, D, GT, kWaves, kStages>(dma, frags, kg, n, rm, c2, first, cnt, ring, qf, q_parts, lane, m_run,
                                              z_run);
      float2 mine;
      if (stats_merge_waves<GT, kWaves, 1>(m_run, z_run, c2, lane, wave, sm.red, mine))
        st_dev_f2(&stat_part[((long long)g * sq.blocks_x + bx) * kRows + threadIdx.x], mine.x, mine.y);
      // published: the partials are device-visible before the head's completion count moves.  The unit's
      // word goes to "done" (2); should a helper and the owner both have run the unit (their partials are
      // bit-identical), only the first to finish counts it.
      drain_vmem();
      __syncthreads();
      if (threadIdx.x == 0) {
        uint32_t* word = &ctl[kCtlUnitA + g * sq.blocks_x + bx];
        if (__hip_atomic_exchange(word, 2u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 2u)
          __hip_atomic_fetch_add(&ctl[kCtlDoneA + g], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
      continue;
    }

    // ------------------------------------------------------------ a score unit
    if (u_b >= a.n_units) break;
    si = seq_of_unit(u_b);
    const SweepSeq sq = a.s[si];
    const int rel = u_b - sq.unit_base;
    g = rel / sq.blocks_x;
    bx = rel % sq.blocks_x;
    const int seq = a.first_seq + si;
    const long long n = sq.n, n_prefix = n - w;
    const char* kg = static_cast<const char*>(a.k) + ((long long)H_kv * sq.tok + (long long)g * n) * T::kRowBytes;
    char* region = a.ws + sq.ws_off;
    const float2* __restrict__ stat_part = reinterpret_cast<const float2*>(region + a.off_stat_part);
    uint32_t* __restrict__ ctl = reinterpret_cast<uint32_t*>(region + a.off_counter);

    const long long n_tiles = (n_prefix + kTileKeys - 1) / kTileKeys;
    const long long t_begin = (long long)bx * sq.tiles_per_block;
    long long t_end = t_begin + sq.tiles_per_block;
    if (t_end > n_tiles) t_end = n_tiles;
    const int n_own = t_begin < t_end ? (int)(t_end - t_begin) : 0;
    const bool halo_left = n_own > 0 && t_begin > 0;
    const bool halo_right = n_own > 0 && t_end < n_tiles;
    const int n_jobs = n_own + (halo_left ? 1 : 0) + (halo_right ? 1 : 0);
    auto job_tile = [&](int j) -> long long {
      if (j < n_own) return t_begin + j;
      return (j == n_own && halo_left) ? t_begin - 1 : t_end;
    };
    __syncthreads();                                   // every wavefront is done with the previous unit's LDS
    // The unit's first tiles are requested before anything else, so that they travel while the head's
    // statistics are awaited and merged.
    q_request(si, g);
    if (threadIdx.x == 0) sm.next_job = kWaves * (kStages - 1);   // published by the barriers below
    int fifo[kStages];
#pragma unroll
    for (int p = 0; p < kStages; ++p) {
      const int j = wave + p * kWaves;
      fifo[p] = (p < kStages - 1 && j < n_jobs) ? j : -1;
    }
    int primed = 0;
#pragma unroll
    for (int p = 0; p < kStages - 1; ++p)
      if (fifo[p] >= 0) {
        dma.issue(kg, job_tile(fifo[p]), n, lane, ring + p * T::kTileChunks);
        ++primed;
      }
    u32x4 qf[GT][kQVec<DT, D>];
    const bool q_parts = q_commit(qf, primed);

    // The head's statistics.  A wait that lasts looks for statistics units of this head nobody has
    // claimed (their owners are not resident yet); one is then run above and this unit set up again.
    if (threadIdx.x == 0) {
      unsigned int spins = 0u;
      int verdict = -1;                                // -1: complete (or gave up), else: span of the unit to run
      while (ld_dev(&ctl[kCtlDoneA + g]) < (unsigned int)sq.blocks_x) {
        __builtin_amdgcn_s_sleep(4);
        ++spins;
        if (spins > a.spin_limit) {
          st_dev(&ctl0[kCtlError], 1u);
          break;
        }
        if ((spins % a.help_after) == 0u) {
          for (int x = 0; x < sq.blocks_x && verdict < 0; ++x) {
            uint32_t* word = &ctl[kCtlUnitA + g * sq.blocks_x + x];
            if (ld_dev(word) == 0u && atomicCAS(word, 0u, 1u) == 0u) verdict = x;
          }
          if (verdict >= 0) break;
        }
      }
      sm.claim[0] = verdict;
    }
    __syncthreads();
    help_bx = sm.claim[0];
    __syncthreads();
    if (help_bx >= 0) {
      help_si = si;
      help_g = g;
      wait_vmcnt<0>();                                 // the tiles requested for this unit have landed; they are asked for again
      __syncthreads();
      continue;
    }
    PoolArgs pa;
    pa.vnorm_part = reinterpret_cast<const float*>(region + a.off_vnorm_part);
    pa.vnorm_blocks = sq.vnorm_blocks;
    pa.pool_half = a.pool_half;
    pa.scores = a.scores + (long long)H_kv * sq.tok;
    pa.vbar = a.vbar + (long long)seq * H_kv;
    pa.token_norm = a.token_norm;
    pa.layer_stat = a.layer_stat + seq;
    pa.ent_part = reinterpret_cast<double2*>(region + a.off_ent_part);
    pa.counters = ctl;
    pa.error_word = &ctl0[kCtlError];
    pa.sel_hist0 = a.sel_ws ? reinterpret_cast<unsigned int*>(a.sel_ws + (size_t)seq * a.sel_stride + a.sel_off_hist) : nullptr;
    pa.plan = a.plan;
    pa.plan_seq = seq;
    float vb = 0.0f;   // this thread's share of the head's value-norm partials (an earlier launch wrote them)
    for (int i = threadIdx.x; i < pa.vnorm_blocks; i += kThreads)
      vb = fmaxf(vb, pa.vnorm_part[(long long)g * pa.vnorm_blocks + i]);
    merge_partials<GT, kWaves, true>((int)threadIdx.x, stat_part + (long long)g * sq.blocks_x * kRows, sq.blocks_x, c2,
                                     sm.sc.merge);
    lds_reads_done();
    __syncthreads();
    write_bias<GT, kWaves>(sm.sc.merge, G < GT ? G : GT, g * G, rm, c2, sm.bias);
    lds_reads_done();
    __syncthreads();
    scores_tiles<DT, D, GT, kWaves, kStages, true, false>(dma, frags, kg, n, n_prefix, c2, t_begin, t_end, n_own, halo_left,
                                                   halo_right, n_jobs, fifo, ring, &sm.next_job, sm.bias, sm.sc.span,
                                                   qf, q_parts, lane, nullptr, 1, rm);
    scores_finish<kThreads>(pa, vb, g, n, n_prefix, w, t_begin, t_end, n_tiles, sm.sc.span, sm.vb, sm.ss, sm.st,
                            &sm.last, (unsigned int)(sq.blocks_x * H_kv), (unsigned int)(g * sq.blocks_x + bx), H_kv,
                            bx == 0, wave, reinterpret_cast<unsigned int*>(&sm.tile[0][0][0]));
    u_b += (int)gridDim.x;
  }
}

// ------------------------------------------------------------------------------------------
// vnorm: per-workgroup maximum over rows of sum_c |V[g, k, c]|, all n rows.  Pure streaming: the
// same direct-to-LDS tile ring as the key sweeps (it sustains more bandwidth than loads into
// registers), 32-row tiles, no matrix work.
// ------------------------------------------------------------------------------------------

template <int DT, int D>
struct VShape {
  static constexpr int kWaves = Tile<DT, D>::kTileBytes > 8192 ? 4 : 8;
  static constexpr int kThreads = kWaves * 64;
  static constexpr int kStagesRaw = (128 * 1024) / (kWaves * Tile<DT, D>::kTileBytes);
  static constexpr int kStages = kStagesRaw > 4 ? 4 : kStagesRaw;
  static_assert(kStages >= 1, "tile too large for the ring");
};

template <int DT, int D>
__global__ void __launch_bounds__((VShape<DT, D>::kThreads))
vnorm_kernel(const SweepArgs a) {
  using T = Tile<DT, D>;
  const SweepSeq sq = a.s[blockIdx.z];
  if (blockIdx.x >= (unsigned int)sq.vnorm_blocks) return;
  const long long n = sq.n;
  const int tiles_per_block = sq.vnorm_tiles_per_block;
  const u32x4* __restrict__ v = static_cast<const u32x4*>(a.v) + (long long)a.H_kv * sq.tok * T::kCpr;
  float* __restrict__ vnorm_part = reinterpret_cast<float*>(a.ws + sq.ws_off + a.off_vnorm_part);
  float* __restrict__ row_norm = a.scores + (long long)a.H_kv * sq.tok;
  uint32_t* __restrict__ counters = reinterpret_cast<uint32_t*>(a.ws + sq.ws_off + a.off_counter);
  const int n_counter_words = kCtlUnitA + a.H_kv * sq.blocks_x;
  constexpr int kWaves = VShape<DT, D>::kWaves;
  constexpr int kStages = VShape<DT, D>::kStages < 2 ? 2 : VShape<DT, D>::kStages;
  __shared__ u32x4 s_tile[kWaves][kStages][T::kTileChunks];
  __shared__ float s_max[kWaves];
  if (blockIdx.x == 0 && blockIdx.y == 0) {
    for (int i = threadIdx.x; i < n_counter_words; i += VShape<DT, D>::kThreads) counters[i] = 0u;
    clear_selection_region(a, (int)blockIdx.z, VShape<DT, D>::kThreads);
  }

  const int lane = threadIdx.x & 63, wave = wave_index();
  const int g = blockIdx.y;
  const char* vg = reinterpret_cast<const char*>(v) + (long long)g * n * T::kRowBytes;
  TileDma<DT, D> dma;
  dma.init(lane);
  FragReader<DT, D> frags;
  frags.init(lane);

  const long long n_tiles = (n + kTileKeys - 1) / kTileKeys;
  const long long t_begin = (long long)blockIdx.x * tiles_per_block;
  long long t_end = t_begin + tiles_per_block;
  if (t_end > n_tiles) t_end = n_tiles;
  const long long first = t_begin + wave;
  const int cnt = first < t_end ? (int)((t_end - first + kWaves - 1) / kWaves) : 0;
  u32x4* ring = s_tile[wave][0];
#pragma unroll
  for (int p = 0; p < kStages - 1; ++p)
    if (p < cnt) dma.issue(vg, first + (long long)p * kWaves, n, lane, ring + p * T::kTileChunks);
  const float best = vnorm_tiles<DT, D, kWaves, kStages, 0>(dma, frags, vg, nullptr, n, first, cnt, 0, 0, ring, lane,
                                                                 a.token_norm != 0, row_norm + (long long)g * n);
  clear_raw_scores(a, sq, g, t_begin, t_end, VShape<DT, D>::kThreads);
  float wave_best = best;
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) wave_best = fmaxf(wave_best, __shfl_xor(wave_best, off));
  if ((threadIdx.x & 63) == 0) s_max[wave] = wave_best;
  __syncthreads();
  if (threadIdx.x == 0) {
    float m = s_max[0];
#pragma unroll
    for (int i = 1; i < kWaves; ++i) m = fmaxf(m, s_max[i]);
    vnorm_part[(long long)g * sq.vnorm_blocks + blockIdx.x] = m;
  }
}

// ------------------------------------------------------------------------------------------
// poolstat: scores[g, i] = Vbar[g] * max_{|i'-i| <= half, i' in prefix} s_raw[g, i'] for the
// prefix, +inf for the window entries; S = sum s, T = sum s ln s in double with a fixed
// reduction order; the last workgroup to finish forms e = (ln S - T / S) / (H_kv * n')  (Eq. 4-5).
// ------------------------------------------------------------------------------------------
constexpr int kPoolThreads = 256;
// Entries per thread: 4 (21013 tokens, 4 heads: 8.5 us; 8: 10.7, the latency of one long workgroup, not bytes), or 8
// where the workspace has no room for the partials of that many workgroups.
constexpr int kPoolPerThread = 8;
constexpr int kPoolChunk = kPoolThreads * kPoolPerThread;

template <int PER>
__global__ void __launch_bounds__(kPoolThreads)
poolstat_kernel(const float* __restrict__ s_raw, long long n, int w, int pool_half, int token_norm,
                const float* __restrict__ vnorm_part, int vnorm_blocks, float* __restrict__ scores,
                float* __restrict__ vbar, float* __restrict__ layer_stat,
                double2* __restrict__ ent_part, uint32_t* __restrict__ counters, unsigned int* __restrict__ sel_hist0,
                const BudgetPlanArgs plan, int plan_seq) {
  __shared__ float s_in[kPoolThreads * PER + 2 * kPoolMaxHalf];
  __shared__ BudgetScratchT<kMaxPlannedLayers> s_plan;
  __shared__ unsigned int s_bins[kSelDigit0Bins];
  const PlanInputs plan_in = plan_prefetch(plan, plan_seq);
  if (sel_hist0 != nullptr)
    for (int i = threadIdx.x; i < kSelDigit0Bins; i += kPoolThreads) s_bins[i] = 0u;      // published by the barrier below
  unsigned int run_digit = 0u, run_len = 0u;
  __shared__ float s_vmax[kPoolThreads / 64];
  __shared__ double s_s[kPoolThreads / 64], s_t[kPoolThreads / 64];
  __shared__ unsigned int s_last;
  const int g = blockIdx.y;
  const long long n_prefix = n - w;
  const long long i0 = (long long)blockIdx.x * kPoolThreads * PER;

  // Vbar of this head from the value-norm partials
  float vb = 0.0f;
  for (int i = threadIdx.x; i < vnorm_blocks; i += kPoolThreads)
    vb = fmaxf(vb, vnorm_part[(long long)g * vnorm_blocks + i]);
  for (int off = 32; off > 0; off >>= 1) vb = fmaxf(vb, __shfl_xor(vb, off));
  if ((threadIdx.x & 63) == 0) s_vmax[threadIdx.x >> 6] = vb;

  for (int i = threadIdx.x; i < kPoolThreads * PER + 2 * pool_half; i += kPoolThreads) {
    const long long p = i0 + i - pool_half;
    s_in[i] = (p >= 0 && p < n_prefix) ? s_raw[(long long)g * n_prefix + p] : -INFINITY;
  }
  __syncthreads();
  vb = s_vmax[0];
  for (int i = 1; i < kPoolThreads / 64; ++i) vb = fmaxf(vb, s_vmax[i]);
  if (blockIdx.x == 0 && threadIdx.x == 0) vbar[g] = vb;

  double acc_s = 0.0, acc_t = 0.0;
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    const int i = j * kPoolThreads + threadIdx.x;
    const long long p = i0 + i;
    if (p < n_prefix) {
      float m = s_in[i + pool_half];
      for (int d = 1; d <= pool_half; ++d) m = fmaxf(m, fmaxf(s_in[i + pool_half - d], s_in[i + pool_half + d]));
      const float s = (token_norm ? scores[(long long)g * n + p] : vb) * m;   // the entry's own value norm, left there by vnorm
      scores[(long long)g * n + p] = s;
      acc_s += (double)s;
      if (s > 0.0f) acc_t += (double)s * (double)logf(s);
      if (sel_hist0 != nullptr) digit0_count(s_bins, s, run_digit, run_len);
    } else if (p < n) {
      scores[(long long)g * n + p] = INFINITY;
      if (sel_hist0 != nullptr) digit0_count(s_bins, INFINITY, run_digit, run_len);
    }
  }
  if (sel_hist0 != nullptr) digit0_flush<kPoolThreads>(s_bins, run_digit, run_len, sel_hist0);
  const bool last = entropy_finish<kPoolThreads>(acc_s, acc_t, ent_part, counters, gridDim.x * gridDim.y,
                                                 blockIdx.y * gridDim.x + blockIdx.x,
                                                 (double)gridDim.y * (double)n_prefix, layer_stat, s_s, s_t, &s_last);
  if (last && plan.e != nullptr) {
    __syncthreads();
    plan_budgets(plan, plan_in, plan_seq, (float)s_t[0], &s_plan);
  }
}

// ------------------------------------------------------------------------------------------ host
static int compute_units() {
  static int cached = 0;
  if (cached == 0) {
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) == hipSuccess &&
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && cus > 0)
      cached = cus;
    else
      cached = 256;   // MI355X
  }
  return cached;
}

int sweep_device_wgs() { return compute_units(); }

int sweep_blocks_per_head(const lava_layer_desc& d) { return d.window > 32 ? 2 : 1; }

int sweep_rows_per_head(const lava_layer_desc& d) {
  // Heads share a block where one block then holds the group: kernels of more blocks would pay for the choice between
  // two sums in their loop (131072 tokens, 32 heads on 8: 1 %), with little left to gain.
  const int heads = d.n_q_heads / d.n_kv_heads;
  if (heads == 2 && d.window <= 16) return 16;
  return (heads == 3 || heads == 4) && d.window <= 8 ? 8 : 32;
}

int sweep_blocks_per_group(const lava_layer_desc& d) {
  const int heads = d.n_q_heads / d.n_kv_heads, share = 32 / sweep_rows_per_head(d);
  return (heads + share - 1) / share * sweep_blocks_per_head(d);
}

bool sweep_has_narrow_shape(const lava_layer_desc& d) { return !(d.dtype == LAVA_F32 && d.head_dim == 128); }

static int sweep_chunk_heads(const lava_layer_desc& d) {
  const int G = sweep_blocks_per_group(d);
  const int gt = d.dtype == LAVA_F32 ? 2 : kMaxChunkHeads;   // f32: query rows as three bf16 parts
  const int heads = G < gt ? G : gt;   // even whenever heads have two blocks: a head's blocks stay in one chunk
  return heads == 3 ? 4 : heads;       // kernels are built for 1, 2 and 4 heads per chunk
}

static int sweep_chunks(const lava_layer_desc& d) {
  const int heads = sweep_chunk_heads(d);
  return (sweep_blocks_per_group(d) + heads - 1) / heads;
}

// A group of two chunks (f32: up to four) can be swept by one workgroup, each chunk by a share of its wavefronts: the
// scores meet in its LDS and it finishes them, and the sequences of a batch share their launches (f32, d_h 128, 8 heads on
// 2, 8 x 1000 tokens: 42 us, one sequence after the other 205).  Apart, a workgroup for each chunk, the scores meet in
// memory, where they have to be cleared first, and a pooling launch finishes them; but a chunk has all wavefronts of a
// workgroup and a short sequence twice or four times the workgroups.  A sequence alone has its group apart where the device
// has few tiles a compute unit (scores and selection, in one workgroup -> apart):
//   two chunks, from 1 tile (below it a span is one round of a chunk's wavefronts, make_sweep_plan) to 10: bf16, d_h 128,
//     40 heads on 8, 9001 tokens 45.9 -> 44.2 us, 14000 51.0 -> 51.5; f32, d_h 64, 32 on 8, 9001 50.9 -> 48.0, 20000 68.5 ->
//     71.4; bf16 to 20 where the KV heads are two and to 28 where there is one (the more workgroups a head has, the more
//     partial statistics each of them merges): scores alone, d_h 128, 12 tiles 40.3 -> 38.0 and 43.6 -> 39.3, at 20 and 28
//     the same; the attention score of one head to 56, since no value rows hide that (28 tiles 63.5 -> 60.3);
//   bf16, two chunks, from 128 on, where spans kept in LDS need several rounds of workgroups: the attention score (40 on 8,
//     204800 tokens, d_h 128 286.6 -> 260.3, d_h 64 191.6 -> 178.5; with d_h 128 from 56: 64 tiles 96.5 -> 95.0, 127 169.6 -> 163.6),
//     the caller's log-sum-exp (135 tiles 155.2 -> 147.7; with d_h 128 from 72: 100 tiles 126.4 -> 112.9, d_h 64 68.7 -> 72.6; below
//     that never: 28 on 4, 9001 28.7 -> 29.8), and one or two KV heads (135 tiles, d_h 64 192 -> 167 and 174 -> 164); not the other
//     scores of more heads (40 on 8, 204800 tokens, d_h 128 354.6 -> 379.8);
//   f32 with d_h 128, of four wavefronts a workgroup, two chunks, up to 5: 8 on 2, 1024 34.9 -> 34.0, 20000 60.7 -> 58.3; 32
//     on 8, 9001 72.9 -> 74.7;
//   three, always (a fourth repeats a head in one workgroup): 12 on 2, 1024 44.7 -> 34.2; 48 on 8, 40000 315 -> 277;
//   four, up to 20: 16 on 2, 1024 44.9 -> 34.5, 40000 110 -> 102; 64 on 8, 20000 175.4 -> 174.5, 40000 316 -> 331.
// (f32 with d_h 64 and more chunks: the same time either way.)
bool sweep_apart(const lava_layer_desc& d, int batch, int64_t n, bool statistics) {
  if (batch > 1) return false;
  const int chunks = sweep_chunks(d);
  const int64_t tiles = (n + kTileKeys - 1) / kTileKeys * d.n_kv_heads, cus = compute_units();
  if (d.dtype == LAVA_F32 && d.head_dim == 128)
    return chunks == 3 || (chunks == 2 && tiles <= 5 * cus) || (chunks == 4 && tiles <= 20 * cus);
  if (chunks != 2) return false;
  if (d.dtype == LAVA_F32) return statistics && tiles > cus && tiles <= 10 * cus;
  if (!statistics) return tiles > (d.head_dim == 128 ? 72 : 128) * cus;
  const bool attention = d.score_kind == LAVA_SCORE_ATTENTION;
  const int64_t few = d.n_kv_heads == 1 ? (attention ? 56 : 28) : d.n_kv_heads == 2 ? 20 : 10;
  if (tiles <= few * cus) return tiles > cus;
  if (attention) return tiles > (d.head_dim == 128 ? 56 : 128) * cus;
  return d.n_kv_heads <= 2 && tiles > 128 * cus;
}

SweepPlan make_sweep_plan(const lava_layer_desc& d, int64_t n, int64_t batch_tokens, bool narrow, bool apart) {
  SweepPlan p;
  p.chunk_heads = sweep_chunk_heads(d);
  const int chunks = sweep_chunks(d);
  // more chunks would leave a wavefront or less to each
  p.wg_chunks = apart ? 1 : chunks == 2 ? 2 : d.dtype != LAVA_F32 ? 1 : chunks > 2 && chunks <= 4 ? 4 : 1;
  p.n_chunks = p.wg_chunks > 1 ? 1 : chunks;
  p.narrow = narrow && sweep_has_narrow_shape(d);
  const int64_t n_tiles = (n + kTileKeys - 1) / kTileKeys;
  // One resident workgroup per slot of the device (one per CU for the wide shape, two for the
  // narrow one): the sweeps keep the group's query rows in registers and a tile ring in LDS, and
  // per-workgroup set-up (query load, partial results) is amortised over as many tiles as possible.
  const int64_t device_wgs = compute_units();
  int64_t target_wgs = p.narrow ? 2 * device_wgs : device_wgs;
  if (tuning().sweep_workgroups > 0) target_wgs = tuning().sweep_workgroups;   // forced by the caller's tuning
  // a sequence that shares its launches with others gets its share of the device, so that the
  // batch as a whole is cut into the longest runs the kernels allow
  const bool shared = batch_tokens > n;
  // (rounded up: a few workgroups too many make the launch a narrow one; without that shape they would be a second round: f32, d_h
  // 128, 12 heads on 2, 35828 + 21654 + 34808 + 42833 tokens, 258 workgroups 437 us, 250 254)
  const auto share = [&](int64_t wgs) {
    return shared ? (wgs * n + (sweep_has_narrow_shape(d) ? batch_tokens - 1 : 0)) / batch_tokens : wgs;
  };
  int64_t max_bx = share(target_wgs) / ((int64_t)d.n_kv_heads * p.n_chunks);
  if (max_bx < 1) max_bx = 1;
  int64_t tpb = (n_tiles + max_bx - 1) / max_bx;
  // Short sequences: spans so short that their tiles and the pooling halo's two are one round of the eight
  // wavefronts (4115 tokens, 8 heads: 16 tiles a workgroup 48.0 us a layer, 8: 44.6, 6: 44.3, 4: 45.4);
  // 32-bit inputs, whose products take several times as long, four (1024 tokens, 2 heads: 16 tiles 69.5 us,
  // 8: 52.0, 6: 48.0, 4: 44.2), or two where the device has the workgroups for it (d_h 64, 1024 tokens 39.1 -> 35.5 us,
  // 4096 41.7 -> 40.1; d_h 128, 8 heads, 1000 tokens 47.7 -> 42.2, 2048 48.9 -> 44.5; three tiles, five with the
  // halo, lose: d_h 64, 9000 tokens 44.5 -> 45.3); and two for the four wavefronts of each of two chunks (bf16, d_h 128,
  // 16 heads on 2, 1024 tokens, scores alone: 21.2 -> 17.6 us, three tiles 18.9).
  const int64_t shortest = d.dtype != LAVA_F32 ? (p.wg_chunks == 2 ? 2 : 6) : (tpb <= 2 ? 2 : 4);
  if (tpb < shortest) tpb = shortest;
  // all heads of a group in one workgroup -> the scores kernel can finish the scores itself, which
  // needs the workgroup's span of raw scores in LDS: a bounded number of tiles per workgroup
  p.fused_pool = p.n_chunks == 1;
  const int64_t fused_cap = p.narrow ? kFusedTilesNarrow : kFusedTilesWide;
  // workgroups that fill whole rounds of `wgs` with spans of at most `cap` tiles
  const auto whole_rounds = [](int64_t tiles, int64_t cap, int64_t wgs) { return (tiles + cap * wgs - 1) / (cap * wgs) * wgs; };
  const int64_t own_tiles = n_tiles * d.n_kv_heads;
  // bounds that hold for either shape, alone or in a batch, and never shrink when n grows: a
  // workspace sized for the longest sequence of a batch must also hold the (differently split)
  // partials of every shorter one
  const int64_t forced = tuning().sweep_workgroups, heads_chunks = (int64_t)d.n_kv_heads * p.n_chunks;
  int64_t bound = (2 * device_wgs > target_wgs ? 2 * device_wgs : target_wgs) / heads_chunks;
  if (bound < 1) bound = 1;
  const auto at_least = [&](int64_t x) { if (bound < x) bound = x; };
  at_least((n_tiles + kFusedTilesNarrow - 1) / kFusedTilesNarrow);
  if (p.fused_pool) {
    at_least(whole_rounds(own_tiles, kFusedTilesWide, forced > 0 ? forced : device_wgs) / d.n_kv_heads);
    at_least(whole_rounds(own_tiles, kFusedTilesNarrow, forced > 0 ? forced : 2 * device_wgs) / d.n_kv_heads);
  }
  p.blocks_x_bound = (int)bound;
  if (p.fused_pool && tpb > fused_cap) {
    // Several rounds of workgroups: the launch as a whole is cut into as many workgroups as fill whole
    // rounds, instead of longest spans whose last round leaves half the device idle (32 sequences of 32768
    // tokens: 2816 workgroups of up to 96 tiles, 5.5 rounds of 512, 1310 us for the whole stack; 3072 of 86,
    // 6 rounds, 1290 us; one of 270000, 28 heads on 4, scores alone: 264 of 128 tiles 368 us, 512 of 66 245).
    const int64_t all = shared ? (batch_tokens + kTileKeys - 1) / kTileKeys * d.n_kv_heads : own_tiles;
    const int64_t fewest = (n_tiles + fused_cap - 1) / fused_cap;
    int64_t bx = n_tiles * whole_rounds(all, fused_cap, target_wgs) / all;
    if (bx > p.blocks_x_bound) bx = p.blocks_x_bound;        // what the workspace holds; at least `fewest`
    if (bx < fewest) bx = fewest;
    tpb = (n_tiles + bx - 1) / bx;
  }
  p.tiles_per_block = (int)tpb;
  p.blocks_x = (int)((n_tiles + tpb - 1) / tpb);
  // value norms: one workgroup per CU for a sequence alone, at least 8 tiles (one per wavefront)
  // each.  Sequences of a batch keep that cut (no share): the kernel's set-up is short, and many
  // small workgroups even out the unequal lengths better than few long ones.
  int64_t vb = (p.narrow ? device_wgs : target_wgs) / d.n_kv_heads;
  if (vb < 1) vb = 1;
  int64_t vtpb = (n_tiles + vb - 1) / vb;
  if (vtpb < 8) vtpb = 8;
  p.vnorm_tiles_per_block = (int)vtpb;
  p.vnorm_blocks = (int)((n_tiles + vtpb - 1) / vtpb);
  const int64_t vb_bound = (target_wgs > device_wgs ? target_wgs : device_wgs) / d.n_kv_heads;
  p.vnorm_blocks_bound = (int)(vb_bound > 1 ? vb_bound : 1);
  if (p.vnorm_blocks_bound < p.blocks_x_bound) p.vnorm_blocks_bound = p.blocks_x_bound;   // value norms cut like the statistics
  return p;
}

int pool_blocks(const lava_layer_desc& d, int64_t n) {
  (void)d;
  return (int)((n + kPoolChunk - 1) / kPoolChunk);
}

// workgroups per KV head whose statistic partials a sequence's workspace region holds
static size_t ent_blocks(const lava_layer_desc& d, int64_t n, const SweepPlan& p) {
  const size_t pool = (size_t)pool_blocks(d, n), sweep = (size_t)p.blocks_x_bound * p.n_chunks;
  return pool > sweep ? pool : sweep;
}

ScoreWorkspace make_score_workspace(const lava_layer_desc& d, int64_t n, bool apart) {
  const SweepPlan p = make_sweep_plan(d, n, 0, false, apart);
  ScoreWorkspace w;
  size_t off = 0;
  w.off_stat_part = off;
  off += align_up(sizeof(float2) * (size_t)d.n_kv_heads * p.n_chunks * p.wg_chunks * p.blocks_x_bound * p.chunk_heads * 32);
  w.off_vnorm_part = off;
  off += align_up(sizeof(float) * (size_t)d.n_kv_heads * p.vnorm_blocks_bound);
  w.off_sraw = off;          // only a group split into chunks goes through raw scores in memory
  if (!p.fused_pool) off += align_up(sizeof(float) * (size_t)d.n_kv_heads * (size_t)(n - d.window));
  w.off_ent_part = off;
  off += align_up(sizeof(double2) * (size_t)d.n_kv_heads * ent_blocks(d, n, p));
  w.off_counter = off;
  off += align_up(sizeof(uint32_t) * ((size_t)kCtlUnitA + (size_t)d.n_kv_heads * p.blocks_x_bound));
  w.bytes = off;
  return w;
}

int32_t launch_vnorm(const lava_layer_desc& d, const SweepArgs& a, int max_vnorm_blocks, hipStream_t s) {
  const dim3 grid(max_vnorm_blocks, d.n_kv_heads, a.n_seq);
  ProfScope ps(KID_VNORM, s);
#define LAVA_VNORM(DTV, DV) \
  hipLaunchKernelGGL((vnorm_kernel<DTV, DV>), grid, dim3(VShape<DTV, DV>::kThreads), 0, s, a)
  if (d.dtype == LAVA_BF16 && d.head_dim == 128) LAVA_VNORM(LAVA_BF16, 128);
  else if (d.dtype == LAVA_BF16 && d.head_dim == 64) LAVA_VNORM(LAVA_BF16, 64);
  else if (d.dtype == LAVA_F32 && d.head_dim == 64) LAVA_VNORM(LAVA_F32, 64);
  else if (d.dtype == LAVA_F32 && d.head_dim == 128) LAVA_VNORM(LAVA_F32, 128);
  else return LAVA_ERR_SHAPE;
#undef LAVA_VNORM
  return launch_status();
}

// Value factor 1.  Where a group is split into chunks the raw scores are cleared too, the heads along y and
// kUnitTiles tiles of each per workgroup: with as few workgroups as the partials take (one, for 4 heads) the clearing was
// the launch (28 heads on 4, attention score: 131072 tokens 147.8 -> 92.6 us for the call, 21013 45.0 -> 36.9).
constexpr int kUnitTiles = 32;
__global__ void __launch_bounds__(256) unit_vnorm_kernel(const SweepArgs a) {
  const SweepSeq sq = a.s[blockIdx.z];
  if (a.n_chunks > 1)
    clear_raw_scores(a, sq, (int)blockIdx.y, (long long)blockIdx.x * kUnitTiles, ((long long)blockIdx.x + 1) * kUnitTiles, 256);
  if (blockIdx.y != 0) return;
  float* vnorm_part = reinterpret_cast<float*>(a.ws + sq.ws_off + a.off_vnorm_part);
  uint32_t* counters = reinterpret_cast<uint32_t*>(a.ws + sq.ws_off + a.off_counter);
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < a.H_kv * sq.vnorm_blocks) vnorm_part[i] = 1.0f;
  for (int j = i; j < kCtlUnitA + a.H_kv * sq.blocks_x; j += (int)gridDim.x * 256) counters[j] = 0u;
  if (blockIdx.x == 0) clear_selection_region(a, (int)blockIdx.z, 256);
}

int32_t launch_unit_vnorm(const lava_layer_desc& d, const SweepArgs& a, int max_vnorm_blocks, hipStream_t s) {
  const int n_part = d.n_kv_heads * max_vnorm_blocks;
  const int n = n_part > kCtlUnitA ? n_part : kCtlUnitA;
  dim3 grid((n + 255) / 256, 1, a.n_seq);
  if (a.n_chunks > 1) {                                        // one sequence per launch
    const unsigned int spans = (unsigned int)((a.s[0].n + kUnitTiles * kTileKeys - 1) / (kUnitTiles * kTileKeys));
    if (spans > grid.x) grid.x = spans;
    grid.y = (unsigned int)d.n_kv_heads;
  }
  ProfScope ps(KID_VNORM, s);
  hipLaunchKernelGGL(unit_vnorm_kernel, grid, dim3(256), 0, s, a);
  return launch_status();
}

float sweep_exp2_scale(const lava_layer_desc& d) {
  const float scale = d.softmax_scale > 0.0f ? d.softmax_scale : 1.0f / sqrtf((float)d.head_dim);
  return scale * kLog2e;
}

// Dispatch over (dtype, head_dim, heads per chunk, chunks per workgroup: several only of the largest).
#define LAVA_SWEEP_DISPATCH(CALL)                                                   \
  do {                                                                              \
    const int gt = p.chunk_heads;                                                   \
    if (d.dtype == LAVA_BF16 && d.head_dim == 128) {                                \
      if (p.wg_chunks == 2) CALL(LAVA_BF16, 128, 4, 2);                             \
      else if (gt == 4) CALL(LAVA_BF16, 128, 4, 1);                                 \
      else if (gt == 2) CALL(LAVA_BF16, 128, 2, 1); else CALL(LAVA_BF16, 128, 1, 1); \
    } else if (d.dtype == LAVA_BF16 && d.head_dim == 64) {                          \
      if (p.wg_chunks == 2) CALL(LAVA_BF16, 64, 4, 2);                              \
      else if (gt == 4) CALL(LAVA_BF16, 64, 4, 1);                                  \
      else if (gt == 2) CALL(LAVA_BF16, 64, 2, 1); else CALL(LAVA_BF16, 64, 1, 1);  \
    } else if (d.dtype == LAVA_F32 && d.head_dim == 64) {                           \
      if (p.wg_chunks == 4) CALL(LAVA_F32, 64, 2, 4);                               \
      else if (p.wg_chunks == 2) CALL(LAVA_F32, 64, 2, 2);                          \
      else if (gt == 2) CALL(LAVA_F32, 64, 2, 1); else CALL(LAVA_F32, 64, 1, 1);    \
    } else if (d.dtype == LAVA_F32 && d.head_dim == 128) {                          \
      if (p.wg_chunks == 4) CALL(LAVA_F32, 128, 2, 4);                              \
      else if (p.wg_chunks == 2) CALL(LAVA_F32, 128, 2, 2);                         \
      else if (gt == 2) CALL(LAVA_F32, 128, 2, 1); else CALL(LAVA_F32, 128, 1, 1);  \
    } else {                                                                        \
      return LAVA_ERR_SHAPE;                                                        \
    }                                                                               \
  } while (0)

int32_t launch_stats(const lava_layer_desc& d, const SweepArgs& a, const SweepPlan& p,
                     bool with_vnorm, hipStream_t s) {
  const dim3 grid(a.n_units);
  ProfScope ps(with_vnorm ? KID_PREPASS : KID_STATS, s);
#define LAVA_STATS_W(DTV, DV, GTV, WV, NCV)                                                                        \
  do {                                                                                                             \
    if (with_vnorm)                                                                                                \
      hipLaunchKernelGGL((stats_kernel<DTV, DV, GTV, WV, true, NCV>), grid, dim3(Shape<DTV, DV, WV>::kThreads), 0, s, a); \
    else                                                                                                           \
      hipLaunchKernelGGL((stats_kernel<DTV, DV, GTV, WV, false, NCV>), grid, dim3(Shape<DTV, DV, WV>::kThreads), 0, s, a); \
  } while (0)
#define LAVA_STATS(DTV, DV, GTV, NCV)                                          \
  do {                                                                         \
    if (Shape<DTV, DV, 4>::kNarrow && p.narrow) LAVA_STATS_W(DTV, DV, GTV, (Shape<DTV, DV, 4>::kNarrow ? 4 : 8), NCV); \
    else LAVA_STATS_W(DTV, DV, GTV, 8, NCV);                                        \
  } while (0)
  LAVA_SWEEP_DISPATCH(LAVA_STATS);
#undef LAVA_STATS
#undef LAVA_STATS_W
  return launch_status();
}

int32_t launch_sweep(const lava_layer_desc& d, const SweepArgs& a, const SweepPlan& p, hipStream_t s) {
  if (!p.fused_pool || p.wg_chunks != 1 || a.lse != nullptr || a.bph != 1 || a.rph != 32) return LAVA_ERR_INVALID_ARG;
  // persistent workgroups: as many as the device keeps resident for this shape, at most one per unit
  const int slots = compute_units() * ((p.narrow && sweep_has_narrow_shape(d)) ? 2 : 1);
  const dim3 grid(a.n_units < slots ? a.n_units : slots);
  ProfScope ps(KID_SWEEP, s);
#define LAVA_SWEEP_W(DTV, DV, GTV, WV) \
  hipLaunchKernelGGL((sweep_kernel<DTV, DV, GTV, WV>), grid, dim3(Shape<DTV, DV, WV>::kThreads), 0, s, a)
#define LAVA_SWEEP(DTV, DV, GTV, NCV)                                          \
  do {                                                                         \
    if (Shape<DTV, DV, 4>::kNarrow && p.narrow) LAVA_SWEEP_W(DTV, DV, GTV, (Shape<DTV, DV, 4>::kNarrow ? 4 : 8)); \
    else LAVA_SWEEP_W(DTV, DV, GTV, 8);                                        \
  } while (0)
  LAVA_SWEEP_DISPATCH(LAVA_SWEEP);
#undef LAVA_SWEEP
#undef LAVA_SWEEP_W
  return launch_status();
}

int32_t launch_scores(const lava_layer_desc& d, const SweepArgs& a, const SweepPlan& p, hipStream_t s) {
  const dim3 grid(a.n_units);
  ProfScope ps(KID_SCORES, s);
#define LAVA_SCORES_W(DTV, DV, GTV, WV, NCV)                                                                \
  do {                                                                                                      \
    if (p.fused_pool)                                                                                       \
      hipLaunchKernelGGL((scores_kernel<DTV, DV, GTV, true, WV, NCV>), grid, dim3(Shape<DTV, DV, WV>::kThreads), \
                         0, s, a);                                                                          \
    else                                                                                                    \
      hipLaunchKernelGGL((scores_kernel<DTV, DV, GTV, false, WV, 1>), grid, dim3(Shape<DTV, DV, WV>::kThreads), \
                         0, s, a);                                                                          \
  } while (0)
#define LAVA_SCORES(DTV, DV, GTV, NCV)                                          \
  do {                                                                          \
    if (Shape<DTV, DV, 4>::kNarrow && p.narrow) LAVA_SCORES_W(DTV, DV, GTV, (Shape<DTV, DV, 4>::kNarrow ? 4 : 8), NCV); \
    else LAVA_SCORES_W(DTV, DV, GTV, 8, NCV);                                        \
  } while (0)
  LAVA_SWEEP_DISPATCH(LAVA_SCORES);
#undef LAVA_SCORES
#undef LAVA_SCORES_W
  return launch_status();
}

int32_t launch_poolstat(const lava_layer_desc& d, int64_t n, const SweepPlan& p, const float* s_raw,
                        const float* vnorm_part, int vnorm_blocks, float* scores, float* vbar,
                        float* layer_stat, double2* ent_part, uint32_t* counters, unsigned int* sel_hist0,
                        const BudgetPlanArgs& plan, int plan_seq, hipStream_t s) {
  const int64_t fine = (n + kPoolThreads * 4 - 1) / (kPoolThreads * 4);
  const bool four = (size_t)fine <= ent_blocks(d, n, p);
  const dim3 grid(four ? (unsigned)fine : (unsigned)pool_blocks(d, n), d.n_kv_heads), block(kPoolThreads);
  ProfScope ps(KID_POOLSTAT, s);
#define LAVA_POOLSTAT(PER)                                                                                        \
  hipLaunchKernelGGL(poolstat_kernel<PER>, grid, block, 0, s, s_raw, (long long)n, d.window, d.pool_kernel / 2,   \
                     d.score_kind == LAVA_SCORE_TOKEN_NORM ? 1 : 0, vnorm_part, vnorm_blocks, scores, vbar,       \
                     layer_stat, ent_part, counters, sel_hist0, plan, plan_seq)
  if (four) LAVA_POOLSTAT(4);
  else LAVA_POOLSTAT(8);
#undef LAVA_POOLSTAT
  return launch_status();
}

}  // namespace lava
