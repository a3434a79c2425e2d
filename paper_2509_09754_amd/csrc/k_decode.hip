// Decode-step attention over the compressed layer cache (Sec. 2 decoding step under the mask of
// Sec. 3): one query token per sequence, the G query heads of a KV group share the group's
// retained rows, which sit packed and variable-length per head as the selection wrote them.
//
//   decode_kernel   one workgroup per "unit" = up to C rows of one head, counted in tiles of 32 rows (the head's
//                   packed rows first, then the rows appended since the eviction: with units of their own, one
//                   appended row cost every head a unit).  Each wavefront streams
//                   32-row tiles: K through its private LDS ring (two tiles ahead), V straight
//                   into registers (one tile ahead; a lane owns the same columns of every row, so
//                   a row is one coalesced load and needs no LDS).  The step is latency-bound
//                   unless enough bytes are in flight per compute unit, and registers are the
//                   larger buffer:
//                     logits   K_tile x Q^T on the matrix cores (the G heads are G columns of the
//                              32-wide operand; the product is exact, accumulation fp32)
//                     softmax  online, in the exp2 domain, per head, kept in the column's lanes
//                     output   acc[head][dims of this lane] += p[key][head] * V[key][dims]: the
//                              probabilities go through LDS as fp32 and are broadcast per key;
//                              V is never rounded or transposed
//                   then the wavefronts' partial (max, sum, acc) are merged.  A head of one unit is
//                   finished there; otherwise the partial goes to the workspace, and the workgroup that
//                   finds all partials of the head published merges them in unit order (deterministic)
//                   and normalises.
//
// A unit's partial is published by a 64-bit flag in the workspace, which the caller hands over with any contents: a flag
// counts only if it equals the call's tag, a number no other call of the process uses (a random start, counted on), and
// whoever merges a head clears its flags, so that the same launch replayed from a graph starts without them.
// There is no counter to clear ahead and no second launch (one layer of 8192 rows: 11.9 us with a merge launch, of
// which it took 5).  Every workgroup stores its flag, waits until the store is visible to the device and then reads the
// flags of its head: whichever store became visible last, its workgroup finds them all.  Should several, each writes
// the same bits.  Nobody waits for another workgroup.
//
// The step is bound by HBM: 2 * d_h * elem bytes per retained row against 4 * G * d_h flop.
#include <math.h>
#include <unistd.h>

#include <atomic>
#include <chrono>

#include "common.h"
#include "tile_ring.h"
#include "xblock.h"

namespace lava {

namespace {

constexpr int kDecWaves = 4;
constexpr int kDecThreads = kDecWaves * 64;

// Two ring stages per wavefront (the K and the V tile of the moment): a workgroup then takes
// well under half of a compute unit's LDS, so two workgroups share a unit and the set-up of one
// overlaps the streaming of the other.
template <int DT, int D>
struct DecShape {
  using T = Tile<DT, D>;
  static constexpr int kStages = 2;
  static constexpr int kBpl = T::kRowBytes / 64;              // bytes of a row one lane owns
  static constexpr int kDpl = kBpl / Elem<DT>::kBytes;        // elements of a row one lane owns
  static_assert(kDpl == 1 || kDpl == 2, "one or two output columns per lane");
  static_assert(kDecWaves * kStages * T::kTileBytes >= kDecWaves * 8 * D * 4, "the ring doubles as the merge buffer");
};

template <int BYTES> struct RawBits;
template <> struct RawBits<2> { using type = unsigned short; };
template <> struct RawBits<4> { using type = unsigned int; };
template <> struct RawBits<8> { using type = uint2; };

// The kDpl elements of a row this lane owns, from their raw bits to floats.
template <int DT, int D>
__device__ __forceinline__ void unpack_v(const typename RawBits<DecShape<DT, D>::kBpl>::type& raw,
                                         float (&x)[DecShape<DT, D>::kDpl]) {
  using S = DecShape<DT, D>;
  if constexpr (DT == LAVA_BF16 && S::kDpl == 1) {
    x[0] = __uint_as_float((unsigned int)raw << 16);
  } else if constexpr (DT == LAVA_BF16) {
    x[0] = __uint_as_float(raw << 16);
    x[1] = __uint_as_float(raw & 0xffff0000u);
  } else if constexpr (S::kDpl == 1) {
    x[0] = __uint_as_float(raw);
  } else {
    x[0] = __uint_as_float(raw.x);
    x[1] = __uint_as_float(raw.y);
  }
}

struct DecodeArgs {
  const u32x4* q;
  const char* k_hat;
  const char* v_hat;
  const long long* head_offsets;   // [batch][H_kv + 1]
  const long long* seq_base;       // [batch] or null
  long long rows_capacity;
  const char* k_tail;
  const char* v_tail;
  long long tail_len, tail_capacity;
  int H, H_kv, G;
  int tiles_per_unit;              // C / 32, a multiple of kDecWaves
  int units_bound;                 // units a sequence can have at most
  int turns;                       // grid: 1 [batch][units_bound], the sequences take turns; 0 [units_bound][batch]
  unsigned int turn_shift, turn_mask;   // unit u of sequence b is in place b - ((u >> shift) & mask) of the sequences' turn
  float c2;                        // softmax scale * log2 e
  float2* part_ml;                 // [batch][units_bound][GP]  (max in log2 units, sum)
  float* part_acc;                 // [batch][units_bound][GP][D]
  unsigned long long* flags;       // [batch][units_bound]  == tag: the unit's partial is published
  unsigned long long tag;
  float* out;                      // [batch][H][D]
  float* lse;                      // [batch][H] or null
};

__device__ __forceinline__ long long ceil_div(long long a, long long b) { return (a + b - 1) / b; }

// Values of a lane both kernels agree on, as scalars (no trip through the LDS unit).
__device__ __forceinline__ unsigned int lane_value(unsigned int x, int lane) {
  return (unsigned int)__builtin_amdgcn_readlane((int)x, lane);
}
__device__ __forceinline__ long long lane_value64(long long x, int lane) {
  const unsigned long long u = (unsigned long long)x;
  return (long long)(((unsigned long long)lane_value((unsigned int)(u >> 32), lane) << 32) | lane_value((unsigned int)u, lane));
}

// The units of one sequence, found by every wavefront on its own with one coalesced load of the
// head offsets: lane g holds head g.  Units are numbered head by head.  Offsets a kernel may follow start at >= 0, never decrease and end
// within the stated capacity; anything else makes `usable` false and nothing is read.
// A decode step over one layer is a chain of dependent trips to memory with the map at its head, so its sums
// and look-ups are lane moves and scalar reads, not shuffles.
struct UnitMap {
  bool usable;
  unsigned int total;        // units of the sequence
  unsigned int incl;         // lane g: units of heads 0..g
  unsigned int cnt;          // lane g: units of head g
  unsigned int packed;       // lane g: tiles of head g's packed rows
  long long off, len;        // lane g: first packed row and number of packed rows of head g
};

template <int CTRL, int ROWS>
__device__ __forceinline__ unsigned int dpp_add(unsigned int x) {
  return x + (unsigned int)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, ROWS, 0xf, false);
}

__device__ __forceinline__ UnitMap map_units(const long long* __restrict__ offs, int n_heads, long long capacity,
                                             int tiles_per_unit, long long tail_len, int lane) {
  UnitMap m;
  const bool head = lane < n_heads;
  const long long o = head ? offs[lane] : 0;
  const long long o_next = head ? offs[lane + 1] : 0;
  const bool bad = (head && (o_next < o || o_next > capacity)) || (lane == 0 && o < 0);
  m.usable = __ballot(bad) == 0ull;
  m.off = o;
  m.len = head && m.usable ? o_next - o : 0;
  const unsigned int tail_tiles = (unsigned int)ceil_div(tail_len, kTileKeys);
  // usable lengths fit 31 bits (capacity and tail < 2^31)
  m.packed = ((unsigned int)m.len + kTileKeys - 1u) / kTileKeys;
  m.cnt = head && m.usable ? (m.packed + tail_tiles + (unsigned int)tiles_per_unit - 1u) / (unsigned int)tiles_per_unit : 0u;
  unsigned int incl = m.cnt;                                 // inclusive sum over the lanes
  incl = dpp_add<0x111, 0xf>(incl);
  incl = dpp_add<0x112, 0xf>(incl);
  incl = dpp_add<0x114, 0xf>(incl);
  incl = dpp_add<0x118, 0xf>(incl);
  incl = dpp_add<0x142, 0xa>(incl);
  incl = dpp_add<0x143, 0xc>(incl);
  m.incl = incl;
  m.total = lane_value(incl, 63);
  return m;
}

// Merge of a head's `mine` units, whose partials start at ml / pa, by a workgroup that has seen all their flags, in unit
// order.  Units are taken kMergeChunk at a time: their (max, sum) pairs go through LDS, every thread then
// knows the chunk's maximum per head without a second trip to memory, and the loads of the partial
// outputs of a whole chunk are independent of each other, so the time does not grow with the
// number of units the way a loop of dependent round trips does.  Across chunks the running result is
// rescaled as in the online softmax.
constexpr int kMergeChunk = 32;
template <int D, int GP>
__device__ __forceinline__ void merge_units(const DecodeArgs& a, int b, int g, int mine, const float2* ml, const float* pa,
                                            float2 (*s_ml)[GP]) {
  constexpr int kPairs = GP * D / 2;                        // outputs in pairs: (t, e) and (t, e + 1)
  constexpr int kOut = (kPairs + kDecThreads - 1) / kDecThreads;
  float M[kOut], L[kOut];
  float2 sum[kOut];
#pragma unroll
  for (int j = 0; j < kOut; ++j) { M[j] = -INFINITY; L[j] = 0.0f; sum[j] = make_float2(0.0f, 0.0f); }
  for (int c0 = 0; c0 < mine; c0 += kMergeChunk) {
    const int nu = mine - c0 < kMergeChunk ? mine - c0 : kMergeChunk;
    float2 pv[kOut][16];                                     // the first sixteen units', on their way beside the pairs
    auto load_units = [&](int u0) {
#pragma unroll
      for (int j = 0; j < kOut; ++j) {
        const int idx = 2 * ((int)threadIdx.x + kDecThreads * j);
        const float2* col = reinterpret_cast<const float2*>(pa + (long long)c0 * GP * D + idx);
#pragma unroll
        for (int u = 0; u < 16; ++u)
          pv[j][u] = idx < GP * D && u0 + u < nu ? ld_dev_f2(&col[(long long)(u0 + u) * (GP * D / 2)]) : make_float2(0.0f, 0.0f);
      }
    };
    load_units(0);
    for (int i = threadIdx.x; i < nu * GP; i += kDecThreads) s_ml[i / GP][i % GP] = ld_dev_f2(&ml[(long long)c0 * GP + i]);
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kOut; ++j) {
      const int t = 2 * ((int)threadIdx.x + kDecThreads * j) / D;
      if (t >= GP) continue;
      float mc = s_ml[0][t].x;
      for (int u = 1; u < nu; ++u) mc = fmaxf(mc, s_ml[u][t].x);
      const float m_new = fmaxf(M[j], mc);                   // finite: a unit holds at least one row
      const float keep = fast_exp2(M[j] - m_new);            // exp2(-inf) = 0 for the first chunk
      M[j] = m_new;
      L[j] *= keep;
      sum[j].x *= keep;
      sum[j].y *= keep;
    }
    for (int u0 = 0; u0 < nu; u0 += 16) {                    // sixteen independent loads per round trip
      if (u0 > 0) load_units(u0);
#pragma unroll
      for (int j = 0; j < kOut; ++j) {
        const int t = 2 * ((int)threadIdx.x + kDecThreads * j) / D;
        if (t >= GP) continue;
#pragma unroll
        for (int u = 0; u < 16; ++u) {                       // unit order: the result does not depend on timing
          if (u0 + u < nu) {
            const float2 st = s_ml[u0 + u][t];
            const float wgt = fast_exp2(st.x - M[j]);
            L[j] += wgt * st.y;
            sum[j].x += wgt * pv[j][u].x;
            sum[j].y += wgt * pv[j][u].y;
          }
        }
      }
    }
    __syncthreads();                                         // the next chunk overwrites s_ml
  }
#pragma unroll
  for (int j = 0; j < kOut; ++j) {
    const int idx = 2 * ((int)threadIdx.x + kDecThreads * j), t = idx / D, e = idx % D;
    if (t >= a.G) continue;
    const long long row = (long long)b * a.H + (long long)g * a.G + t;
    a.out[row * D + e] = sum[j].x / L[j];
    a.out[row * D + e + 1] = sum[j].y / L[j];
    if (a.lse != nullptr && e == 0) a.lse[row] = (M[j] + log2f(L[j])) * 0.6931471805599453f;
  }
}

// What the units do not write: zeros for heads without rows, NaN everywhere if the offsets cannot be followed.
// By one workgroup of the sequence.
template <int D>
__device__ __forceinline__ void fill_heads(const DecodeArgs& a, int b, const UnitMap& um, bool bad) {
  if (!bad && __ballot((int)(threadIdx.x & 63) < a.H_kv && um.cnt == 0u) == 0ull) return;   // the same in every wavefront
  for (int g = 0; g < a.H_kv; ++g) {
    if (!bad && lane_value(um.cnt, g) != 0u) continue;
    const long long row0 = (long long)b * a.H + (long long)g * a.G;
    for (int i = threadIdx.x; i < a.G * D; i += kDecThreads) a.out[row0 * D + i] = bad ? NAN : 0.0f;
    if (a.lse != nullptr && (int)threadIdx.x < a.G) a.lse[row0 + threadIdx.x] = bad ? NAN : -INFINITY;
  }
}

template <int DT, int D, int GP>
__global__ void __launch_bounds__(kDecThreads) decode_kernel(DecodeArgs a) {
  using S = DecShape<DT, D>;
  using T = Tile<DT, D>;
  constexpr int kStages = S::kStages;
  constexpr int kDpl = S::kDpl;
  __shared__ u32x4 s_tile[kDecWaves][kStages][T::kTileChunks];   // after the sweep: float [kDecWaves][GP][D]
  constexpr int kPs = GP < 4 ? 4 : GP;                      // floats per key in s_p (one or two 128-bit reads)
  __shared__ __attribute__((aligned(16))) float s_p[kDecWaves][kTileKeys + 1][kPs];   // probabilities; row 32: rescale factors
  __shared__ float s_m[kDecWaves][GP], s_l[kDecWaves][GP];

  const int lane = threadIdx.x & 63, wave = wave_index();
  // Sequences take turns, their first units before their second ones: the workgroups without a unit then come last, and the
  // others spread evenly over the XCDs, which get every eighth workgroup each (turned from unit to unit where the number of
  // sequences would have a sequence's units on few of the XCDs).
  unsigned int unit = blockIdx.x;
  int b = blockIdx.y;
  if (a.turns) {                                            // uniform
    unit = blockIdx.y;
    b = (int)blockIdx.x + (int)((unit >> a.turn_shift) & a.turn_mask);
    if (b >= (int)gridDim.x) b -= (int)gridDim.x;
  }
  const UnitMap um = map_units(a.head_offsets + (long long)b * (a.H_kv + 1), a.H_kv, a.rows_capacity,
                               a.tiles_per_unit, a.tail_len, lane);
  const bool bad = !um.usable || um.total > (unsigned int)a.units_bound;
  if (unit == 0u) fill_heads<D>(a, b, um, bad);
  if (bad || unit >= um.total) return;                      // uniform: nothing to follow, or no such unit
  const int g = __builtin_ctzll(__ballot(um.incl > unit));
  const long long u = (long long)unit - ((long long)lane_value(um.incl, g) - (long long)lane_value(um.cnt, g));
  const long long packed_tiles = lane_value(um.packed, g);
  const long long off_g = lane_value64(um.off, g), len_g = lane_value64(um.len, g);
  const long long tail_tiles = ceil_div(a.tail_len, kTileKeys);
  const long long first_tile = u * a.tiles_per_unit;         // of the head's tiles: packed ones, then appended ones
  const long long packed_at = ((a.seq_base ? a.seq_base[b] : (long long)b * a.rows_capacity) + off_g) * T::kRowBytes;
  const long long tail_at = ((long long)b * a.H_kv + g) * a.tail_capacity * T::kRowBytes;
  long long n_tiles = packed_tiles + tail_tiles - first_tile;
  if (n_tiles > a.tiles_per_unit) n_tiles = a.tiles_per_unit;
  // Tile i of this wavefront: which rows (of the packed ones or of the appended ones), as a tile index there, and how many
  // rows there are
  struct Src {
    bool packed;
    long long tile, rows;
  };

  // This wavefront's tiles: wave, wave + kDecWaves, ...  Vector-memory operations complete in issue
  // order and the K ring is awaited by count, so the order below is part of the protocol:
  //   K_0, K_1 | query rows, V_0 | then per tile i:  K_{i+2} ... V_{i+1}
  using VRaw = typename RawBits<S::kBpl>::type;
  TileDma<DT, D> dma;
  dma.init(lane);
  const int cnt = wave < n_tiles ? (int)((n_tiles - wave + kDecWaves - 1) / kDecWaves) : 0;
  u32x4* ring = s_tile[wave][0];
  FragReader<DT, D> frags;
  frags.init_at(lane, lds_addr(ring));
  const unsigned int p_addr = lds_addr(&s_p[wave][0][0]);
  auto source = [&](int i) -> Src {
    const long long t = first_tile + wave + (long long)i * kDecWaves;
    return t < packed_tiles ? Src{true, t, len_g} : Src{false, t - packed_tiles, a.tail_len};
  };
  auto issue_k = [&](int i) {
    const Src src = source(i);
    dma.issue(src.packed ? a.k_hat + packed_at : a.k_tail + tail_at, src.tile, src.rows, lane, ring + (i % kStages) * T::kTileChunks);
  };
  const unsigned int v_lane = (unsigned int)lane * S::kBpl;   // a row is a uniform address plus this
  auto load_v = [&](VRaw (&dst)[kTileKeys], int i) {
    const Src src = source(i);
    const long long row0 = src.tile * kTileKeys;
    const char* p = (src.packed ? a.v_hat + packed_at : a.v_tail + tail_at) + row0 * T::kRowBytes;
    if (row0 + kTileKeys <= src.rows) {
#pragma unroll
      for (int kk = 0; kk < kTileKeys; ++kk) dst[kk] = *reinterpret_cast<const VRaw*>(p + kk * T::kRowBytes + v_lane);
    } else {                                                // rows beyond the last one repeat it
      const int last = (int)(src.rows - 1 - row0);          // 0 .. 30, uniform
#pragma unroll
      for (int kk = 0; kk < kTileKeys; ++kk)
        dst[kk] = *reinterpret_cast<const VRaw*>(p + (kk < last ? kk : last) * T::kRowBytes + v_lane);
    }
  };
  if (cnt > 0) issue_k(0);
  if (cnt > 1) issue_k(1);
  asm volatile("" ::: "memory");

  // the group's query rows as the 32-column operand: column t < G is head g*G + t
  const int col = lane & 31, half = lane >> 5;
  u32x4 qf[T::kSteps];
#pragma unroll
  for (int j = 0; j < T::kSteps; ++j) {
    u32x4 x = u32x4{0u, 0u, 0u, 0u};
    if (col < a.G) x = a.q[((long long)b * a.H + (long long)g * a.G + col) * T::kCpr + 2 * j + half];
    qf[j] = x;
  }
  const unsigned int p_col = p_addr + (unsigned int)(col * 4);                  // row 0 of s_p, this head's column
  const unsigned int p_mine = p_col + (unsigned int)(4 * half * kPs * 4);       // first key this lane's results cover
  VRaw v0[kTileKeys], v1[kTileKeys];
  if (cnt > 0) load_v(v0, 0);

  float m_run = -INFINITY, l_run = 0.0f;                    // of head `col` (lanes col < G)
  float acc[GP][kDpl];
#pragma unroll
  for (int t = 0; t < GP; ++t)
#pragma unroll
    for (int e = 0; e < kDpl; ++e) acc[t][e] = 0.0f;

  // PAR = it % 2 is the ring stage of K_it
  auto step = [&](auto par, int it, VRaw (&v_cur)[kTileKeys], VRaw (&v_next)[kTileKeys]) {
    constexpr int PAR = decltype(par)::value;
    // ---------------- K tile: logits, online softmax, probabilities to LDS
    {
      // everything older than V_it (32 loads) and, if it was requested, K_{it+1} has landed
      if (it + 1 < cnt) wait_vmcnt<T::kLoads + kTileKeys>(); else wait_vmcnt<kTileKeys>();
      u32x4 kf[T::kSteps];
      frags.template read_at<PAR * T::kTileBytes>(kf);      // in registers on return: the stage is free
      if (it + 2 < cnt) issue_k(it + 2);
      asm volatile("" ::: "memory");
      // two independent accumulation chains halve the latency of the dependent MFMAs
      f32x16 x = {0}, x2 = {0};
#pragma unroll
      for (int j = 0; j < T::kSteps; j += 2) {
        x = mfma_chunk<DT>(kf[j], qf[j], x);
        x2 = mfma_chunk<DT>(kf[j + 1], qf[j + 1], x2);
      }
      x += x2;                                              // x[v]: key 8*(v/4) + 4*half + v%4, head col
      const Src src = source(it);
      const long long left = src.rows - src.tile * kTileKeys;   // rows from this tile on (uniform)
      float mt = -INFINITY;
      if (left >= kTileKeys) {
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          x[v] *= a.c2;
          mt = fmaxf(mt, x[v]);
        }
      } else {                                              // a partial tile
        int h4 = 4 * half;
        asm volatile("" : "+v"(h4));                        // keeps this path's temporaries out of the hot loop
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const float s = (h4 + 8 * (v / 4) + (v % 4) < (int)left) ? x[v] * a.c2 : -INFINITY;
          x[v] = s;
          mt = fmaxf(mt, s);
        }
      }
      mt = fmaxf(mt, __shfl_xor(mt, 32));
      const float m_new = fmaxf(m_run, mt);                 // finite: a tile holds at least one row
      const float alpha = fast_exp2(m_run - m_new);
      float ls = 0.0f;
      if (col < GP) {
        static_for<16>([&](auto vc) {
          constexpr int v = decltype(vc)::value;
          const float p = fast_exp2(x[v] - m_new);
          ls += p;
          lds_write32_at<(8 * (v / 4) + (v % 4)) * kPs * 4>(p_mine, p);
        });
        if (half == 0) lds_write32_at<kTileKeys * kPs * 4>(p_col, alpha);
      }
      l_run = l_run * alpha + ls;
      m_run = m_new;
    }
    lds_reads_done();                                       // LDS operations of a wavefront execute in order
    // ---------------- V tile (already requested): request the next one, rescale, accumulate
    {
      if (it + 1 < cnt) load_v(v_next, it + 1);
      asm volatile("" ::: "memory");
      u32x4 al[kPs / 4];
      static_for<kPs / 4>([&](auto cc) {
        constexpr int c = decltype(cc)::value;
        lds_read128_at<(kTileKeys * kPs + 4 * c) * 4>(p_addr, al[c]);
      });
#pragma unroll
      for (int t = 0; t < GP; ++t)
#pragma unroll
        for (int e = 0; e < kDpl; ++e) acc[t][e] *= __uint_as_float(al[t / 4][t % 4]);
      // probabilities of four keys per read batch
      static_for<kTileKeys / 4>([&](auto kc) {
        constexpr int k4 = 4 * decltype(kc)::value;
        u32x4 pr[kPs / 4][4];
        static_for<kPs / 4>([&](auto cc) {
          constexpr int c = decltype(cc)::value;
          lds_read128x4_strided<kPs * 4, (k4 * kPs + 4 * c) * 4>(p_addr, pr[c][0], pr[c][1], pr[c][2], pr[c][3]);
        });
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
          float vx[kDpl];
          unpack_v<DT, D>(v_cur[k4 + kk], vx);
#pragma unroll
          for (int t = 0; t < GP; ++t) {
            const float p = __uint_as_float(pr[t / 4][kk][t % 4]);
#pragma unroll
            for (int e = 0; e < kDpl; ++e) acc[t][e] = fmaf(p, vx[e], acc[t][e]);
          }
        }
        // pin the accumulators here: otherwise the multiply-adds of all batches sink below the reads
        // of all batches, which then have to stay in registers together
#pragma unroll
        for (int t = 0; t < GP; ++t)
#pragma unroll
          for (int e = 0; e < kDpl; ++e) asm volatile("" : "+v"(acc[t][e]));
      });
    }
  };
  int it = 0;
  for (; it + 1 < cnt; it += 2) {
    step(std::integral_constant<int, 0>{}, it, v0, v1);
    step(std::integral_constant<int, 1>{}, it + 1, v1, v0);
  }
  if (it < cnt) step(std::integral_constant<int, 0>{}, it, v0, v1);
  wait_vmcnt<0>();

  // ---------------- merge the wavefronts of the unit
  l_run += __shfl_xor(l_run, 32);
  if (lane < GP) {
    s_m[wave][lane] = m_run;
    s_l[wave][lane] = l_run;
  }
  __syncthreads();                                          // every wavefront is done with its ring
  float (*s_acc)[GP][D] = reinterpret_cast<float (*)[GP][D]>(&s_tile[0][0][0]);
#pragma unroll
  for (int t = 0; t < GP; ++t)
#pragma unroll
    for (int e = 0; e < kDpl; ++e) s_acc[wave][t][lane * kDpl + e] = acc[t][e];
  __syncthreads();
  const int mine = (int)lane_value(um.cnt, g);               // units of the head
  const long long slot = (long long)b * a.units_bound + unit;
  constexpr int kPairs = GP * D / 2;
#pragma unroll
  for (int j = 0; j < (kPairs + kDecThreads - 1) / kDecThreads; ++j) {
    const int idx = 2 * ((int)threadIdx.x + kDecThreads * j), t = idx / D, e = idx % D;
    if (t >= GP) continue;
    float M = s_m[0][t];
#pragma unroll
    for (int w2 = 1; w2 < kDecWaves; ++w2) M = fmaxf(M, s_m[w2][t]);
    float L = 0.0f;
    float2 sum = make_float2(0.0f, 0.0f);
#pragma unroll
    for (int w2 = 0; w2 < kDecWaves; ++w2) {
      const float wgt = fast_exp2(s_m[w2][t] - M);
      L += wgt * s_l[w2][t];
      sum.x += wgt * s_acc[w2][t][e];
      sum.y += wgt * s_acc[w2][t][e + 1];
    }
    if (mine > 1) {
      st_dev_f2(reinterpret_cast<float2*>(a.part_acc + slot * GP * D + idx), sum.x, sum.y);
      if (e == 0) st_dev_f2(&a.part_ml[slot * GP + t], M, L);
    } else if (t < a.G) {
      const long long row = (long long)b * a.H + (long long)g * a.G + t;
      a.out[row * D + e] = sum.x / L;
      a.out[row * D + e + 1] = sum.y / L;
      if (a.lse != nullptr && e == 0) a.lse[row] = (M + log2f(L)) * 0.6931471805599453f;
    }
  }
  if (mine <= 1) return;
  // ---------------- publish the unit; merge the head if all its units are published
  drain_vmem();
  __syncthreads();                                          // every thread's share of the partial is visible to the device
  unsigned long long* flags = a.flags + slot - u;           // of the head's units
  int* s_all = reinterpret_cast<int*>(&s_p[0][0][0]);
  if (wave == 0) {
    if (lane == 0) {
      st_dev(&flags[u], a.tag);
      drain_vmem();
    }
    bool all = true;
    for (int i = lane; i < mine; i += 64) all &= ld_dev(&flags[i]) == a.tag;
    const bool every = __ballot(!all) == 0ull;
    if (lane == 0) *s_all = every ? 1 : 0;
  }
  __syncthreads();
  if (*s_all == 0) return;
  for (int i = threadIdx.x; i < mine; i += kDecThreads) st_dev(&flags[i], 0ull);
  static_assert(sizeof(s_tile) >= kMergeChunk * GP * sizeof(float2), "the ring is the merge's buffer");
  merge_units<D, GP>(a, b, g, mine, a.part_ml + (slot - u) * GP, a.part_acc + (slot - u) * GP * D,
                     reinterpret_cast<float2 (*)[GP]>(&s_tile[0][0][0]));
}

template <int DT, int D, int GP>
int32_t launch_one(const DecodeArgs& a, int batch, hipStream_t s) {
  ProfScope ps(KID_DECODE, s);
  hipLaunchKernelGGL((decode_kernel<DT, D, GP>), a.turns ? dim3(batch, a.units_bound) : dim3(a.units_bound, batch), dim3(kDecThreads), 0, s, a);
  return launch_status();
}

// A number that no other call of this process uses and that memory holds by chance once in 2^64 words: a mixed
// counter (a bijection of 64 bits) from a start of its own in every process.  The mixing and the counter's step are
// those of SplitMix64 (Steele, Lea, Flood, "Fast splittable pseudorandom number generators", 2014).
unsigned long long mix64(unsigned long long x) {
  x = (x ^ (x >> 30)) * 0xbf58476d1ce4e5b9ull;
  x = (x ^ (x >> 27)) * 0x94d049bb133111ebull;
  return x ^ (x >> 31);
}
unsigned long long next_tag() {
  static std::atomic<unsigned long long> next{
      mix64((unsigned long long)std::chrono::steady_clock::now().time_since_epoch().count() ^
            ((unsigned long long)getpid() << 40) ^ (unsigned long long)reinterpret_cast<uintptr_t>(&next))};
  for (;;) {
    const unsigned long long tag = mix64(next.fetch_add(0x9e3779b97f4a7c15ull, std::memory_order_relaxed));
    if (tag != 0ull) return tag;                            // 0 is "not published"
  }
}

int padded_group(int G) { return G <= 1 ? 1 : G <= 2 ? 2 : G <= 4 ? 4 : 8; }

int device_cus() {
  static int cus = 0;
  if (cus == 0) {
    int dev = 0, n = 0;
    if (hipGetDevice(&dev) == hipSuccess &&
        hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && n > 0)
      cus = n;
    else
      return 256;
  }
  return cus;
}

}  // namespace

DecodePlan make_decode_plan(const lava_layer_desc& d, int32_t batch, int64_t rows_capacity, int64_t tail_len) {
  DecodePlan p;
  const int64_t step = kTileKeys * kDecWaves;
  const int64_t tail_tiles = (tail_len + kTileKeys - 1) / kTileKeys;
  const int64_t total = (int64_t)batch * (rows_capacity + (int64_t)d.n_kv_heads * tail_tiles * kTileKeys);
  // Rows per unit: the units should fill whole rounds of the workgroups the device holds at a time (two per compute unit; one
  // with rows of 512 bytes, whose ring takes 128 KB of LDS), with as few units as that allows (every unit pays its set-up and
  // leaves a partial result to merge).  A head is expected to waste half a unit; a sequence of one head wastes what it does.
  // One round (12 x 32768 rows on 8 KV heads: 896 rows a unit, one round, 40.8 us, 512, two, 44.1; f32 128.2 -> 95.9 with
  // 896, which is two rounds there) if its units are no longer than one and a half heads (of 256 rows, two: 32 KV heads, 12 x
  // 4096: 10.2, with 128 14.4) and no longer than 1280 rows or a quarter of a head: the last ones end unevenly by as much
  // (7 heads a group, 24 x 32768: 1920, one round, 104.7, 896, two, 94.3).
  // bf16 with d_h 64, of which four workgroups share a compute unit, so that one round of two leaves half the wavefronts
  // out: 256 rows or an eighth of a head (4 KV heads, 16 x 8192: 384, one round, 16.2, 256, two, 15.5).
  // Heads of many units are merged by one workgroup each, about 0.11 us a unit, where 128 more rows in a unit are 1.6 us: no
  // fewer than the root of 8 rows a head (one head of 32768 rows: 128 39.3, 512 23.4; of 100000: 256 61.9, 896 35.7).
  const bool small = d.head_dim == 64 && d.dtype == LAVA_BF16;
  const int64_t one_round = small ? 256 : 1280, per_head = small ? 8 : 4, most = 16 * step;
  const bool one_per_cu = d.head_dim == 128 && d.dtype == LAVA_F32;
  const int64_t resident = (one_per_cu ? 1 : 2) * (int64_t)device_cus();
  const int64_t heads = (int64_t)batch * d.n_kv_heads;
  const auto units = [&](int64_t rows) {
    if (d.n_kv_heads == 1) return batch * ((rows_capacity + tail_tiles * kTileKeys + rows - 1) / rows);
    return total / rows + heads / 2;
  };
  int64_t rounds = (units(most) + resident - 1) / resident, c;
  if (rounds < 1) rounds = 1;
  for (;; ++rounds) {
    for (c = step; c < most && units(c) > rounds * resident; c += step) {}
    if (rounds > 1 || c == step || (c == 2 * step && c * heads <= 2 * total) ||
        (2 * c * heads <= 3 * total && (c <= one_round || per_head * c * heads <= total)))
      break;
  }
  const int64_t merged = (int64_t)(sqrt(8.0 * (double)total / (double)heads) / step + 0.5) * step;
  if (c < merged) c = merged < most ? merged : most;
  if (tuning().decode_rows_per_unit >= step) c = tuning().decode_rows_per_unit / step * step;   // caller's tuning
  p.rows_per_unit = (int)c;
  p.group_pad = padded_group(d.n_q_heads / d.n_kv_heads);
  // a head's last packed tile, and its last unit, may be partial
  const int64_t tiles = (rows_capacity + kTileKeys - 1) / kTileKeys + d.n_kv_heads * (1 + tail_tiles);
  p.units_bound = (tiles + c / kTileKeys - 1) / (c / kTileKeys) + d.n_kv_heads;
  if (p.units_bound < 1) p.units_bound = 1;
  // Sequences take turns (48 x 8192 rows on 2 KV heads, 487 units for 512 places: 60.5 us one sequence after the other, 46.3
  // in turn; f32, d_h 128, 100 x 1024 on 1, two units and two idle workgroups a sequence: 63 and 36), unless two workgroups
  // share a compute unit, few are idle and a sixteenth of the last round's places is free: there is little to gain then, and
  // rows at the same distance in every sequence are read together (64 x 8192, 939 units: 64.6 and 66.7; 16 x 8192, 405: 20.3
  // and 20.9).
  const int64_t filled = units(c), last = (filled + resident - 1) / resident;
  const bool even = !one_per_cu && 16 * filled <= 15 * last * resident && 10 * filled >= 7 * batch * p.units_bound;
  p.turns = batch > 1 && !even && p.units_bound <= 65535;     // the units are the grid's y then
  const size_t slots = (size_t)batch * (size_t)p.units_bound * p.group_pad;
  p.off_ml = 0;
  p.off_acc = align_up(slots * sizeof(float2));
  p.off_flags = p.off_acc + align_up(slots * d.head_dim * sizeof(float));
  p.bytes = p.off_flags + align_up((size_t)batch * (size_t)p.units_bound * sizeof(unsigned long long));
  return p;
}

int32_t launch_decode(const lava_layer_desc& d, int32_t batch, const void* q, const void* k_hat,
                      const void* v_hat, const int64_t* head_offsets, const int64_t* seq_base,
                      int64_t rows_capacity, const void* k_tail, const void* v_tail, int64_t tail_len,
                      int64_t tail_capacity, float* out, float* lse, void* ws, const DecodePlan& p,
                      hipStream_t s) {
  DecodeArgs a;
  a.q = static_cast<const u32x4*>(q);
  a.k_hat = static_cast<const char*>(k_hat);
  a.v_hat = static_cast<const char*>(v_hat);
  a.head_offsets = reinterpret_cast<const long long*>(head_offsets);
  a.seq_base = reinterpret_cast<const long long*>(seq_base);
  a.rows_capacity = rows_capacity;
  a.k_tail = static_cast<const char*>(k_tail);
  a.v_tail = static_cast<const char*>(v_tail);
  a.tail_len = tail_len;
  a.tail_capacity = tail_capacity;
  a.H = d.n_q_heads;
  a.H_kv = d.n_kv_heads;
  a.G = d.n_q_heads / d.n_kv_heads;
  a.tiles_per_unit = p.rows_per_unit / kTileKeys;
  a.units_bound = (int)p.units_bound;
  a.turns = p.turns ? 1 : 0;
  // A workgroup's place among those of its unit and all before it, modulo 8, is its XCD.  An odd batch moves a sequence on by
  // itself; an even one of eight and more by one place a unit; two, four and six cover their XCDs first.
  const unsigned int even = (unsigned int)batch & (0u - (unsigned int)batch);   // largest power of two that divides it
  a.turn_shift = batch >= 8 || even == 1u ? 0u : even == 2u ? 2u : 1u;
  a.turn_mask = even == 1u ? 0u : batch >= 8 ? 7u : even - 1u;
  const float scale = d.softmax_scale > 0.0f ? d.softmax_scale : 1.0f / sqrtf((float)d.head_dim);
  a.c2 = scale * kLog2e;
  a.part_ml = reinterpret_cast<float2*>(static_cast<char*>(ws) + p.off_ml);
  a.part_acc = reinterpret_cast<float*>(static_cast<char*>(ws) + p.off_acc);
  a.flags = reinterpret_cast<unsigned long long*>(static_cast<char*>(ws) + p.off_flags);
  a.tag = next_tag();
  a.out = out;
  a.lse = lse;

#define LAVA_DECODE_CASE(DT, D, GP) \
  if (d.dtype == DT && d.head_dim == D && p.group_pad == GP) return launch_one<DT, D, GP>(a, batch, s);
#define LAVA_DECODE_GROUPS(DT, D) \
  LAVA_DECODE_CASE(DT, D, 1) LAVA_DECODE_CASE(DT, D, 2) LAVA_DECODE_CASE(DT, D, 4) LAVA_DECODE_CASE(DT, D, 8)
  LAVA_DECODE_GROUPS(LAVA_BF16, 128)
  LAVA_DECODE_GROUPS(LAVA_BF16, 64)
  LAVA_DECODE_GROUPS(LAVA_F32, 128)
  LAVA_DECODE_GROUPS(LAVA_F32, 64)
#undef LAVA_DECODE_GROUPS
#undef LAVA_DECODE_CASE
  return LAVA_ERR_SHAPE;
}

}  // namespace lava
