// Wavefront-private tile ring shared by the kernels that stream a cache through the matrix cores.
//
// A 32-row tile of one head is a contiguous span of HBM.  It travels HBM -> LDS with coalesced
// 128-bit direct-to-LDS loads (no staging registers) into a ring of XOR-swizzled buffers owned by
// one wavefront, several tiles ahead of the one being consumed; arrival of a tile is a vmcnt wait
// that leaves the younger tiles in flight, so a sweep needs no workgroup barrier.  The tile is
// then read in MFMA operand layout.
//
// MFMA 32x32 layouts (wave64): operand lane l supplies row/column l%32 and k-slice l/32; result
// register v of lane l is element (8*(v/4) + 4*(l/32) + v%4, l%32).
#pragma once

#include <hip/hip_runtime.h>

#include <utility>

#include "common.h"

namespace lava {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));   // 16 bytes held in registers

constexpr float kLog2e = 1.4426950408889634f;

template <int DT> struct Elem;
template <> struct Elem<LAVA_BF16> { static constexpr int kBytes = 2; };
template <> struct Elem<LAVA_F32> { static constexpr int kBytes = 4; };

// acc += A(8 values of k) x B(8 values of k).  Both operands use the same lane -> k mapping, so
// any fixed assignment of a row's elements to (step, lane half) gives the full dot product.
__device__ __forceinline__ f32x16 mfma_bf16(const u32x4& a, const u32x4& b, f32x16 acc) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), acc, 0, 0, 0);
}

// the same over 16 bytes of either type, 32-bit values through the 32-bit instructions
template <int DT>
__device__ __forceinline__ f32x16 mfma_chunk(const u32x4& a, const u32x4& b, f32x16 acc) {
  if constexpr (DT == LAVA_BF16) {
    return mfma_bf16(a, b, acc);
  } else {
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.x), __uint_as_float(b.x), acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.y), __uint_as_float(b.y), acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.z), __uint_as_float(b.z), acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.w), __uint_as_float(b.w), acc, 0, 0, 0);
    return acc;
  }
}

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// x of this lane + x of lane ^ 32, without a trip through the LDS unit
__device__ __forceinline__ float add_halves(float x) {
  const auto h = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(h[0]) + __uint_as_float(h[1]);
}

#define LAVA_GLOBAL_AS __attribute__((address_space(1)))
#define LAVA_LDS_AS __attribute__((address_space(3)))

// Wait until at most N vector-memory operations of this wavefront are still outstanding.  Loads
// complete in issue order, so this guarantees every load older than the N youngest has landed.
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  static_assert(N >= 0 && N < 64, "vmcnt is a 6-bit counter");
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt((N & 0xF) | (0x7 << 4) | (0xF << 8) | ((N >> 4) << 14));
  asm volatile("" ::: "memory");
}

// (m1, z1) (+) (m2, z2) for sums of exp2((x - m) * c2); empty sets are (-inf, 0).
__device__ __forceinline__ void merge_stat(float& m, float& z, float m2, float z2, float c2) {
  const float mn = fmaxf(m, m2);
  const float f1 = (m == mn) ? 1.0f : fast_exp2((m - mn) * c2);
  const float f2 = (m2 == mn) ? 1.0f : fast_exp2((m2 - mn) * c2);
  z = z * f1 + z2 * f2;
  m = mn;
}

// (m, z) (+) p[0] (+) ... (+) p[N - 1], the maximum first: N independent exponentials instead of a chain of them.
template <int N>
__device__ __forceinline__ void merge_stats(const float2 (&p)[N], float c2, float& m, float& z) {
  float mn = m;
#pragma unroll
  for (int i = 0; i < N; ++i) mn = fmaxf(mn, p[i].x);
  z *= m == mn ? 1.0f : fast_exp2((m - mn) * c2);
#pragma unroll
  for (int i = 0; i < N; ++i) z += p[i].y * (p[i].x == mn ? 1.0f : fast_exp2((p[i].x - mn) * c2));
  m = mn;
}

template <int DT, int D>
struct Tile {
  static constexpr int kRowBytes = D * Elem<DT>::kBytes;
  static constexpr int kCpr = kRowBytes / 16;          // 16-byte chunks per row
  static constexpr int kSteps = kCpr / 2;              // chunk steps (two lane halves per step)
  static constexpr int kLoads = kTileKeys * kCpr / 64; // 128-bit loads per lane per tile
  static constexpr int kTileChunks = kTileKeys * kCpr;
  static constexpr int kTileBytes = kTileKeys * kRowBytes;
};

// Direct-to-LDS reads of 32-key tiles into a ring stage.  Instruction i moves 1 KiB: lane l lands
// at chunk slot i*64 + l of the stage, i.e. row (i*64+l)/kCpr, slot s = (i*64+l)%kCpr, and fetches
// the row's chunk s ^ (row & 7): the swizzle is applied on the global side because the LDS side
// of such a load is linear.  The per-lane byte offsets inside a tile are computed once; a full tile
// is then (wave-uniform tile address) + (per-lane offset), which needs no vector arithmetic.
template <int DT, int D>
struct TileDma {
  using T = Tile<DT, D>;
  static constexpr int kRowsPerLoad = 64 / T::kCpr;                                // rows one instruction covers
  static constexpr int kVariants = kRowsPerLoad >= 8 ? 1 : 8 / kRowsPerLoad;        // distinct (row & 7) patterns
  unsigned int loff[kVariants];   // per-lane byte offset inside the 1 KiB slice of load i, variant i % kVariants

  __device__ __forceinline__ void init(int lane) {
#pragma unroll
    for (int i = 0; i < kVariants; ++i) {
      const int q = i * 64 + lane;
      const int row = q / T::kCpr, slot = q % T::kCpr;
      loff[i] = (unsigned int)((row - i * kRowsPerLoad) * T::kRowBytes + ((slot ^ (row & 7)) << 4));
    }
  }

  // Every row of the tile exists.  Load i covers bytes [i KiB, (i+1) KiB) of the tile on both sides;
  // the common part of the offset is an instruction immediate (< 4 KiB) applied to the global and
  // the LDS address alike, plus a scalar 4 KiB step, so a load costs no vector arithmetic.
  __device__ __forceinline__ void issue_full(const char* __restrict__ tile_base, u32x4* stage) const {
#pragma unroll
    for (int i = 0; i < T::kLoads; ++i) {
      const char* src = tile_base + (i / 4) * 4096 + loff[i % kVariants];
      u32x4* dst = stage + (i / 4) * 256;
      switch (i % 4) {
        case 0: __builtin_amdgcn_global_load_lds((const LAVA_GLOBAL_AS void*)src, (LAVA_LDS_AS void*)dst, 16, 0, 0); break;
        case 1: __builtin_amdgcn_global_load_lds((const LAVA_GLOBAL_AS void*)src, (LAVA_LDS_AS void*)dst, 16, 1024, 0); break;
        case 2: __builtin_amdgcn_global_load_lds((const LAVA_GLOBAL_AS void*)src, (LAVA_LDS_AS void*)dst, 16, 2048, 0); break;
        default: __builtin_amdgcn_global_load_lds((const LAVA_GLOBAL_AS void*)src, (LAVA_LDS_AS void*)dst, 16, 3072, 0); break;
      }
    }
  }

  // rows at or beyond n are read from row n - 1 (callers mask or drop them)
  __device__ __forceinline__ void issue_clamped(const char* __restrict__ head_base, long long tile,
                                                long long n, int lane, u32x4* stage) const {
    // This path runs once per sweep.  The lane index goes through an opaque move so that nothing
    // derived from it is computed ahead of the hot loop and kept in registers across it.
    asm volatile("" : "+v"(lane));
    const char* tile_base = head_base + tile * T::kTileBytes;
    const int last = (int)(n - 1 - tile * kTileKeys);      // last existing row of the tile, 0 .. 30
#pragma unroll
    for (int i = 0; i < T::kLoads; ++i) {
      const int q = i * 64 + lane;
      const int row = q / T::kCpr, slot = q % T::kCpr;
      const int src_row = row < last ? row : last;
      const char* src = tile_base + (unsigned int)(src_row * T::kRowBytes + ((slot ^ (row & 7)) << 4));
      __builtin_amdgcn_global_load_lds((const LAVA_GLOBAL_AS void*)src, (LAVA_LDS_AS void*)(stage + i * 64), 16,
                                       0, 0);
    }
  }

  __device__ __forceinline__ void issue(const char* __restrict__ head_base, long long tile, long long n,
                                        int lane, u32x4* stage) const {
    if ((tile + 1) * kTileKeys <= n) {
      issue_full(head_base + tile * T::kTileBytes, stage);
    } else {
      issue_clamped(head_base, tile, n, lane, stage);
    }
  }
};

// Wait for the oldest tile of a ring while `younger` (0 .. kMaxRingStages-1) tiles stay in flight.
constexpr int kMaxRingStages = 4;
template <int DT, int D>
__device__ __forceinline__ void wait_tile(int younger) {
  using T = Tile<DT, D>;
  switch (younger) {
    case 0: wait_vmcnt<0>(); break;
    case 1: wait_vmcnt<T::kLoads>(); break;
    case 2: wait_vmcnt<2 * T::kLoads>(); break;
    default: wait_vmcnt<3 * T::kLoads>(); break;
  }
}

// ------------------------------------------------------------------------------------------
// LDS accesses written as instructions.
//
// While direct-to-LDS loads are in flight the compiler cannot tell which LDS bytes they will
// write, so before EVERY ordinary LDS access it waits for all of them (vmcnt(0)), which turns the
// ring into one tile in flight per wavefront.  The ring protocol already guarantees that a stage
// is only read after its own loads have landed (wait_tile) and only refilled after its reads have
// returned (lds_reads_done), so the LDS accesses inside a sweep are issued as instructions the
// compiler does not reason about.  Each read helper ends with its own wait: its results are valid
// on return.  Addresses are LDS byte offsets (lds_addr).
// ------------------------------------------------------------------------------------------
__device__ __forceinline__ unsigned int lds_addr(const void* p) {
  return (unsigned int)(unsigned long long)(LAVA_LDS_AS const char*)p;
}

// every LDS operation this wavefront has issued is complete
__device__ __forceinline__ void lds_reads_done() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

__device__ __forceinline__ void lds_read128x4(unsigned int a0, unsigned int a1, unsigned int a2, unsigned int a3,
                                              u32x4& o0, u32x4& o1, u32x4& o2, u32x4& o3) {
  asm volatile(
      "ds_read_b128 %0, %4\n\t"
      "ds_read_b128 %1, %5\n\t"
      "ds_read_b128 %2, %6\n\t"
      "ds_read_b128 %3, %7\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(o0), "=&v"(o1), "=&v"(o2), "=&v"(o3)
      : "v"(a0), "v"(a1), "v"(a2), "v"(a3)
      : "memory");
}

// Offsets known at compile time travel in the instruction (16-bit field), so that one address
// register serves every access of a loop instead of one hoisted register per access.
// four reads at byte offsets OFF, OFF + STRIDE, OFF + 2*STRIDE, OFF + 3*STRIDE from one address
template <int STRIDE, int OFF = 0>
__device__ __forceinline__ void lds_read128x4_strided(unsigned int a, u32x4& o0, u32x4& o1, u32x4& o2, u32x4& o3) {
  static_assert(OFF >= 0 && OFF + 3 * STRIDE < 65536, "LDS instruction offset field");
  asm volatile(
      "ds_read_b128 %0, %4 offset:%5\n\t"
      "ds_read_b128 %1, %4 offset:%6\n\t"
      "ds_read_b128 %2, %4 offset:%7\n\t"
      "ds_read_b128 %3, %4 offset:%8\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(o0), "=&v"(o1), "=&v"(o2), "=&v"(o3)
      : "v"(a), "n"(OFF), "n"(OFF + STRIDE), "n"(OFF + 2 * STRIDE), "n"(OFF + 3 * STRIDE)
      : "memory");
}

// four reads at one compile-time offset from four addresses
template <int OFF>
__device__ __forceinline__ void lds_read128x4_at(unsigned int a0, unsigned int a1, unsigned int a2, unsigned int a3,
                                                 u32x4& o0, u32x4& o1, u32x4& o2, u32x4& o3) {
  static_assert(OFF >= 0 && OFF < 65536, "LDS instruction offset field");
  asm volatile(
      "ds_read_b128 %0, %4 offset:%8\n\t"
      "ds_read_b128 %1, %5 offset:%8\n\t"
      "ds_read_b128 %2, %6 offset:%8\n\t"
      "ds_read_b128 %3, %7 offset:%8\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(o0), "=&v"(o1), "=&v"(o2), "=&v"(o3)
      : "v"(a0), "v"(a1), "v"(a2), "v"(a3), "n"(OFF)
      : "memory");
}

template <int OFF>
__device__ __forceinline__ void lds_read128_at(unsigned int a, u32x4& o) {
  static_assert(OFF >= 0 && OFF < 65536, "LDS instruction offset field");
  asm volatile("ds_read_b128 %0, %1 offset:%2\n\ts_waitcnt lgkmcnt(0)" : "=&v"(o) : "v"(a), "n"(OFF) : "memory");
}

template <int OFF>
__device__ __forceinline__ void lds_write32_at(unsigned int a, float x) {
  static_assert(OFF >= 0 && OFF < 65536, "LDS instruction offset field");
  asm volatile("ds_write_b32 %0, %1 offset:%2" : : "v"(a), "v"(x), "n"(OFF) : "memory");
}

// f(std::integral_constant<int, 0>{}), ..., f(std::integral_constant<int, N - 1>{}): a loop whose
// index is a constant expression inside the body
template <int... I, class F>
__device__ __forceinline__ void static_for_impl(std::integer_sequence<int, I...>, F&& f) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
  static_for_impl(std::make_integer_sequence<int, N>{}, f);
}

__device__ __forceinline__ void lds_read128(unsigned int a, u32x4& o) {
  asm volatile("ds_read_b128 %0, %1\n\ts_waitcnt lgkmcnt(0)" : "=&v"(o) : "v"(a) : "memory");
}

// *a += 1 in LDS, returns the value before.  Call from ONE lane.
__device__ __forceinline__ unsigned int lds_fetch_inc(unsigned int a) {
  unsigned int v;
  const unsigned int one = 1u;
  asm volatile("ds_add_rtn_u32 %0, %1, %2\n\ts_waitcnt lgkmcnt(0)" : "=&v"(v) : "v"(a), "v"(one) : "memory");
  return v;
}

__device__ __forceinline__ void lds_write64(unsigned int a, float2 x) {
  asm volatile("ds_write_b64 %0, %1" : : "v"(a), "v"(x) : "memory");
}
__device__ __forceinline__ float2 lds_read64(unsigned int a) {
  float2 x;
  asm volatile("ds_read_b64 %0, %1\n\ts_waitcnt lgkmcnt(0)" : "=&v"(x) : "v"(a) : "memory");
  return x;
}

__device__ __forceinline__ void lds_write32(unsigned int a, float x) {
  asm volatile("ds_write_b32 %0, %1" : : "v"(a), "v"(x) : "memory");
}

// *a = max(*a, x) for values that are not negative, which order as integers
__device__ __forceinline__ void lds_max32(unsigned int a, float x) {
  asm volatile("ds_max_u32 %0, %1" : : "v"(a), "v"(x) : "memory");
}

// Per-lane addresses of a tile's MFMA operand fragments: lane l holds row l % 32 and, at step j,
// the row's 16-byte chunk 2j + l/32 (stored at slot chunk ^ (row & 7)).
template <int DT, int D>
struct FragReader {
  using T = Tile<DT, D>;
  unsigned int foff[T::kSteps];

  __device__ __forceinline__ void init(int lane) {
    const int row = lane & 31, half = lane >> 5;
#pragma unroll
    for (int j = 0; j < T::kSteps; ++j) foff[j] = (unsigned int)((row * T::kCpr + ((2 * j + half) ^ (row & 7))) << 4);
  }

  // Variant for a ring whose stage is known at compile time: init_at folds the ring's address into
  // the per-lane offsets once, read_at<OFF> then needs no address arithmetic at all.
  __device__ __forceinline__ void init_at(int lane, unsigned int ring) {
    init(lane);
#pragma unroll
    for (int j = 0; j < T::kSteps; ++j) foff[j] += ring;
  }
  template <int OFF>
  __device__ __forceinline__ void read_at(u32x4 (&frag)[T::kSteps]) const {
#pragma unroll
    for (int j = 0; j < T::kSteps; j += 4)
      lds_read128x4_at<OFF>(foff[j], foff[j + 1], foff[j + 2], foff[j + 3], frag[j], frag[j + 1], frag[j + 2],
                            frag[j + 3]);
  }

  // `stage`: LDS byte address of the ring stage.  The fragments are in registers on return.
  __device__ __forceinline__ void read(unsigned int stage, u32x4 (&frag)[T::kSteps]) const {
    static_assert(T::kSteps % 4 == 0, "fragments are read four at a time");
#pragma unroll
    for (int j = 0; j < T::kSteps; j += 4)
      lds_read128x4(stage + foff[j], stage + foff[j + 1], stage + foff[j + 2], stage + foff[j + 3], frag[j],
                    frag[j + 1], frag[j + 2], frag[j + 3]);
  }
};

// The matrix cores take 32 query rows at a time, a row block.  A head whose window has more than 32 rows is
// handled as `bph` = 2 row blocks: block index hb = head * 2 + block, rows block * 32 ..; a group of two heads with
// windows of at most 16 rows, or of up to four with at most 8, is one block, `rph` = 16 or 8 rows a head: with a block of
// its own such a head pays matrix instructions, exponentials, normalisers and query rows for 32 (1024 tokens, 8 heads on
// 2, 8 rows, f32: 32.0 -> 28.5 us a layer).
// Everything up to the point where a head's window rows are summed treats a row block as a head.
struct RowMap {
  int heads;     // query heads per KV group
  int G;         // row blocks per KV group
  int bph;       // row blocks per head: 1 or 2
  int rph;       // rows per head in a block: 32, 16 or 8
  int w;         // window rows
};
struct RowAt {
  int head, row;   // query head of the layer, window row
  bool real;       // the head exists and has that row
};
// Row r (0 .. 31) of row block hb, blocks counted through the KV groups.  BLOCKS: of the kernel's group; heads can share
// a block only where that is the whole group (the choice costs the other kernels a us of set-up).
template <int BLOCKS>
__device__ __forceinline__ RowAt row_at(const RowMap& m, int hb, int r) {
  RowAt x;
  if (BLOCKS > 1 || m.rph == 32) {                             // uniform
    x.head = hb / m.bph;
    x.row = (hb % m.bph) * 32 + r;
    x.real = x.row < m.w;
  } else {
    const int g = hb / m.G, h = ((hb - g * m.G) * 32 + r) / m.rph;
    x.head = g * m.heads + h;
    x.row = r & (m.rph - 1);
    x.real = h < m.heads && x.row < m.w;
  }
  return x;
}

// Query rows as a wavefront keeps them for a sweep: the 16-byte chunks of FragReader (bf16), or for every pair of
// chunks their three bf16 parts (f32, see split8).
template <int DT, int D> constexpr int kQVec = DT == LAVA_BF16 ? Tile<DT, D>::kSteps : Tile<DT, D>::kSteps / 2 * 3;

// 32-bit values as sums of three bf16: x = hi + mid + lo, exactly (8 + 8 + 8 bits, each part what is nearest to what
// the parts before it leave; 32-bit products of such parts: Henry, Tang, Heinecke, "Leveraging the bfloat16 artificial
// intelligence datatype for higher-precision computations", 2019).  `a` and `b`: four values each.
__device__ __forceinline__ unsigned int pack_bf16(float lo, float hi) {
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  return __builtin_bit_cast(unsigned int, __builtin_convertvector((f32x2{lo, hi}), bf16x2));
}
__device__ __forceinline__ float bf16_low(unsigned int u) { return __uint_as_float(u << 16); }
__device__ __forceinline__ float bf16_high(unsigned int u) { return __uint_as_float(u & 0xffff0000u); }
__device__ __forceinline__ void split8(const u32x4& a, const u32x4& b, u32x4& hi, u32x4& mid, u32x4& lo) {
  const unsigned int x[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float x0 = __uint_as_float(x[2 * i]), x1 = __uint_as_float(x[2 * i + 1]);
    hi[i] = pack_bf16(x0, x1);
    const float r0 = x0 - bf16_low(hi[i]), r1 = x1 - bf16_high(hi[i]);
    mid[i] = pack_bf16(r0, r1);
    lo[i] = pack_bf16(r0 - bf16_low(mid[i]), r1 - bf16_high(mid[i]));
  }
}
// The same for any values: hi is cut instead, so that it does not overflow, and infinities and NaN are a first part only.
__device__ __forceinline__ void split8_any(const u32x4& a, const u32x4& b, u32x4& hi, u32x4& mid, u32x4& lo) {
  const unsigned int x[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    unsigned int h[2];
    float r[2];
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const unsigned int u = x[2 * i + e];
      const bool special = (u & 0x7f800000u) == 0x7f800000u;
      h[e] = (u & 0xffff0000u) | (special && (u & 0x007fffffu) != 0u ? 0x00400000u : 0u);   // a NaN stays one
      r[e] = special ? 0.0f : __uint_as_float(u) - __uint_as_float(h[e]);
    }
    hi[i] = __builtin_amdgcn_perm(h[1], h[0], 0x07060302u);
    mid[i] = pack_bf16(r[0], r[1]);
    lo[i] = pack_bf16(r[0] - bf16_low(mid[i]), r[1] - bf16_high(mid[i]));
  }
}
// A NaN does not count.
__device__ __forceinline__ float abs_max8(const u32x4& a, const u32x4& b, float m) {
  const unsigned int x[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
#pragma unroll
  for (int i = 0; i < 8; i += 2) m = fmaxf(fmaxf(m, fabsf(__uint_as_float(x[i]))), fabsf(__uint_as_float(x[i + 1])));
  return m;
}
// Products of parts stand for products of values where both are below this: no part, product of parts or sum of 128
// products overflows, which with parts of either sign would give a NaN for a product that is infinite (a key that the
// type's lowest value masks, a query of 2^24 and more), and a part that is lost below the smallest normal values (2^-126)
// changes a product by less than 2^-66.
constexpr float kPartsLimit = 1152921504606846976.0f;            // 2^60

// A head's query rows from their chunks.  Returns true if products of their parts may be used (f32; the parts add up to
// the value either way).
template <int DT, int D>
__device__ __forceinline__ bool make_q(const u32x4 (&raw)[Tile<DT, D>::kSteps], u32x4 (&q)[kQVec<DT, D>]) {
  if constexpr (DT == LAVA_BF16) {
#pragma unroll
    for (int j = 0; j < Tile<DT, D>::kSteps; ++j) q[j] = raw[j];
    return true;
  } else {
    float top = 0.0f;
#pragma unroll
    for (int j = 0; j < Tile<DT, D>::kSteps; j += 2) top = abs_max8(raw[j], raw[j + 1], top);
    const bool parts = top < kPartsLimit;
    if (__ballot(!parts) == 0ull) {                              // uniform
#pragma unroll
      for (int j = 0; j < Tile<DT, D>::kSteps; j += 2)
        split8(raw[j], raw[j + 1], q[j / 2 * 3], q[j / 2 * 3 + 1], q[j / 2 * 3 + 2]);
    } else {
#pragma unroll
      for (int j = 0; j < Tile<DT, D>::kSteps; j += 2)
        split8_any(raw[j], raw[j + 1], q[j / 2 * 3], q[j / 2 * 3 + 1], q[j / 2 * 3 + 2]);
    }
    return parts;
  }
}

// Query fragments of the chunk's row blocks hb0 .. hb0 + nh - 1, one copy per wavefront straight from
// global memory: row r = lane % 32 of the block (zero beyond the window or the chunk).  Returns this lane's share of
// "products of parts may be used".
template <int DT, int D, int GT>
__device__ __forceinline__ bool load_q(const u32x4* __restrict__ qg, int hb0, int nh, const RowMap& rm, int lane,
                                       u32x4 (&qf)[GT][kQVec<DT, D>]) {
  using T = Tile<DT, D>;
  const int r = lane & 31, half = lane >> 5;
  bool parts = true;
#pragma unroll
  for (int t = 0; t < GT; ++t) {
    const RowAt at = row_at<GT>(rm, hb0 + t, r);
    u32x4 raw[T::kSteps];
#pragma unroll
    for (int j = 0; j < T::kSteps; ++j) {
      u32x4 x = u32x4{0u, 0u, 0u, 0u};
      if (t < nh && at.real) x = qg[((long long)at.head * rm.w + at.row) * T::kCpr + 2 * j + half];
      raw[j] = x;
    }
    parts &= make_q<DT, D>(raw, qf[t]);
  }
  return parts;
}

// Row block hb of the chunk hb0 .. hb0 + nh - 1 as a tile in LDS, requested with direct-to-LDS loads by one
// wavefront: no registers, and the block is read once per workgroup.  Rows beyond the window repeat its last
// one, blocks beyond the chunk its last block: their results are masked or never used.
template <int DT, int D, int BLOCKS>
__device__ __forceinline__ void request_q(const TileDma<DT, D>& dma, const u32x4* __restrict__ qg, int hb0, int nh, int t,
                                          const RowMap& rm, int lane, u32x4* buf) {
  using T = Tile<DT, D>;
  const int hb = hb0 + (t < nh ? t : nh - 1);
  const char* q = reinterpret_cast<const char*>(qg);
  if (BLOCKS > 1 || rm.rph == 32) {                            // uniform: one head's rows, which follow each other
    const int head = hb / rm.bph, row0 = (hb % rm.bph) * 32;
    dma.issue_clamped(q + ((long long)head * rm.w + row0) * T::kRowBytes, 0, rm.w - row0 < 32 ? rm.w - row0 : 32, lane, buf);
    return;
  }
  const int g = hb / rm.G, h0 = (hb - g * rm.G) * (32 / rm.rph);
#pragma unroll
  for (int i = 0; i < T::kLoads; ++i) {
    const int c = i * 64 + lane, r = c / T::kCpr, slot = c % T::kCpr;
    int h = h0 + r / rm.rph, row = r & (rm.rph - 1);
    h = h < rm.heads ? h : rm.heads - 1;
    row = row < rm.w ? row : rm.w - 1;
    const char* src = q + ((long long)(g * rm.heads + h) * rm.w + row) * T::kRowBytes + ((slot ^ (r & 7)) << 4);
    __builtin_amdgcn_global_load_lds((const LAVA_GLOBAL_AS void*)src, (LAVA_LDS_AS void*)(buf + i * 64), 16, 0, 0);
  }
}

// One head's 32 x 32 block of raw dot products: keys x rows (KEYS_AS_ROWS) or rows x keys.
template <int D, bool KEYS_AS_ROWS>
__device__ __forceinline__ f32x16 dot_tile(const u32x4 (&kf)[Tile<LAVA_BF16, D>::kSteps],
                                           const u32x4 (&qh)[Tile<LAVA_BF16, D>::kSteps]) {
  f32x16 acc = {0};
#pragma unroll
  for (int j = 0; j < Tile<LAVA_BF16, D>::kSteps; ++j)
    acc = KEYS_AS_ROWS ? mfma_bf16(kf[j], qh[j], acc) : mfma_bf16(qh[j], kf[j], acc);
  return acc;
}

// The same for 32-bit inputs and all heads of a chunk at once.  The 32-bit matrix instruction has a sixteenth of the
// bf16 rate, so values are taken as three bf16 parts and six of the nine products summed: hi*hi on its own, the small
// ones together, and then the two sums, by an addition that rounds to nearest where the matrix unit cuts.  What is left
// out (mid*lo, lo*mid, lo*lo) is below 0.99 * 2^-24 of a product of the values.  Error of the logits against 64 bits, in
// 2^-24 of the logit, where one channel makes the row (all roundings add up): largest 2.0, rms 0.45; 32-bit instructions
// 1.3 and 0.44 (hi cut instead of rounded and one sum: 5.2 and 0.60; with mid*lo and lo*mid: 1.3 and 0.44, sweeps 12 %
// longer).  Of the scores of normally distributed rows of 128 channels: largest 1.0e-6, rms 3.4e-7; 32-bit instructions
// 2.4e-6 and 3.9e-7.
// Bound by the vector unit: a tile of 32 keys and 128 values takes 48 bf16 instructions of 32 cycles per head (32-bit:
// 64 of 64 cycles), the split 350 vector instructions of 5 cycles, shared by two heads (more do not fit the registers).
// Scores of a layer of 9001 tokens, 32 heads on 8: 72.7 -> 61.6 us; 1024 tokens of 64 values, 8 heads on 2: 22.8 -> 16.5.
// Tiles or queries with large values or infinities (kPartsLimit) go through the 32-bit instructions, query rows put
// together again; a NaN's parts are NaN.
template <int D, int GT, bool KEYS_AS_ROWS>
__device__ __forceinline__ void dot_tiles(const u32x4 (&kf_in)[Tile<LAVA_F32, D>::kSteps],
                                          const u32x4 (&qf)[GT][kQVec<LAVA_F32, D>], bool q_parts, f32x16 (&acc)[GT]) {
  constexpr int kPairs = Tile<LAVA_F32, D>::kSteps / 2;
  u32x4 kf[2 * kPairs];
#pragma unroll
  for (int j = 0; j < 2 * kPairs; ++j) kf[j] = kf_in[j];
  float top = 0.0f;
#pragma unroll
  for (int j = 0; j < kPairs; ++j) top = abs_max8(kf[2 * j], kf[2 * j + 1], top);
#pragma unroll
  for (int t = 0; t < GT; ++t) acc[t] = f32x16{0};
  auto mul = [&](const u32x4& k, const u32x4& q, f32x16& sum) {
    sum = KEYS_AS_ROWS ? mfma_bf16(k, q, sum) : mfma_bf16(q, k, sum);
  };
  if (q_parts && __ballot(!(top < kPartsLimit)) == 0ull) {
    u32x4 hi[kPairs];
    f32x16 small[GT];
#pragma unroll
    for (int t = 0; t < GT; ++t) small[t] = f32x16{0};
#pragma unroll
    for (int j = 0; j < kPairs; ++j) {
      u32x4 mid, lo;
      split8(kf[2 * j], kf[2 * j + 1], hi[j], mid, lo);
      // the next pair's split begins here: with all of them in front of the products the query rows leave the vector
      // registers and are copied back for every tile (160 moves, 5 % of the time)
      if (j + 1 < kPairs) asm volatile("" : "+v"(kf[2 * j + 2]), "+v"(kf[2 * j + 3]), "+v"(hi[j]), "+v"(mid), "+v"(lo));
#pragma unroll
      for (int t = 0; t < GT; ++t) mul(lo, qf[t][3 * j], small[t]);
#pragma unroll
      for (int t = 0; t < GT; ++t) mul(hi[j], qf[t][3 * j + 2], small[t]);
#pragma unroll
      for (int t = 0; t < GT; ++t) mul(mid, qf[t][3 * j + 1], small[t]);
#pragma unroll
      for (int t = 0; t < GT; ++t) mul(mid, qf[t][3 * j], small[t]);
#pragma unroll
      for (int t = 0; t < GT; ++t) mul(hi[j], qf[t][3 * j + 1], small[t]);
    }
#pragma unroll
    for (int j = 0; j < kPairs; ++j)
#pragma unroll
      for (int t = 0; t < GT; ++t) mul(hi[j], qf[t][3 * j], acc[t]);
#pragma unroll
    for (int t = 0; t < GT; ++t)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[t][v] += small[t][v];
  } else {
#pragma unroll
    for (int j = 0; j < 2 * kPairs; ++j)
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int t = 0; t < GT; ++t) {
          const int at = (j & 1) * 2 + i / 2;
          unsigned int part[3] = {qf[t][j / 2 * 3][at], qf[t][j / 2 * 3 + 1][at], qf[t][j / 2 * 3 + 2][at]};
          asm volatile("" : "+v"(part[0]), "+v"(part[1]), "+v"(part[2]));   // or they are put together ahead of the sweep's loop
          // the second and third part first: with the first, the second one could overflow at the largest values
          const float q = (i & 1) ? bf16_high(part[0]) + (bf16_high(part[1]) + bf16_high(part[2]))
                                  : bf16_low(part[0]) + (bf16_low(part[1]) + bf16_low(part[2]));
          const float k = __uint_as_float(kf[j][i]);
          acc[t] = KEYS_AS_ROWS ? __builtin_amdgcn_mfma_f32_32x32x2f32(k, q, acc[t], 0, 0, 0)
                                : __builtin_amdgcn_mfma_f32_32x32x2f32(q, k, acc[t], 0, 0, 0);
        }
  }
}

// Index of the wavefront inside its workgroup as a scalar, so that everything derived from it
// (tile numbers, ring stages, loop bounds) stays in scalar registers and scalar branches.
__device__ __forceinline__ int wave_index() { return __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)); }

}  // namespace lava
