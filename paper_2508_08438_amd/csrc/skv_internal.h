// Internal definitions shared by the translation units of libskv (host + device).
#ifndef SKV_INTERNAL_H
#define SKV_INTERNAL_H

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "skv.h"

#define SKV_HD __host__ __device__

// ---- flattened tree as the kernels see it -------------------------------------------------
// Blocks of one node are contiguous in every per-block array ("flat block index").
// Node 0 is the root (no blocks).  A node's children are found through an open-addressed
// table keyed by a 64-bit hash of the child's whole first block; a hit is always confirmed
// by comparing the 16 tokens, so results never depend on the hash.
struct SkvNode {       // 16 bytes
  int32_t first;       // flat index of the node's first block
  int32_t n_blocks;    // blocks on the compressed edge
  int32_t tab_off;     // first slot of the child table (in SkvSlot units)
  int32_t tab_cap;     // slots (power of two), 0 = leaf
};
struct SkvSlot {       // 16 bytes
  uint32_t hash_lo, hash_hi;
  int32_t child;       // node index, -1 = empty, -2 = removed (probing goes on)
  int32_t pad;
};
// Per-block counters, one plane of uint32 per field: 0 hit_cur, 1..4 tenant bitmap, 5 hit_pre, 6 u_pre, 7 predicate streak.
// Planes and not records: the blocks of a path are contiguous, so the atomics of a wavefront on one field fall into two or
// three cache lines, where 32-byte records took sixteen (4096 lookups, 0.77 M matched blocks: 69.6 us with records, 34.4
// with planes, 29 without any atomics).
#define SKV_CTR_FIELDS 8

struct SkvTreeDev {
  const int32_t* tok;     // [n_blocks][16]
  const int32_t* page;    // [n_blocks]   address vector
  int32_t* meta;          // [n_blocks]   bit31 = private_tag, bits 0..30 = creator_id (demotion sets bit31)
  const int32_t* canon;   // [n_blocks]   input block id that created the entry
  const int32_t* flat_of; // [n_in_blocks] flat index of the entry an input block created, -1 if none
  uint32_t* ctr;          // [SKV_CTR_FIELDS][ctr_plane]
  size_t ctr_plane;       // blocks the slab has room for
  uint32_t* epoch;        // [n_blocks]   epoch counter value at the block's last access
  uint32_t* limits;       // [1] SKV_LIMIT_* bits of the limits the branching lookup has run into since the last read
  const SkvNode* nodes;   // [n_nodes+1]
  const SkvSlot* slots;
  int32_t n_blocks, n_nodes, n_tenants, n_pages;  // n_blocks: block records in use, evicted ones (canon < 0) included
  uint32_t cur_epoch;     // stamped on every block a lookup matches
};

struct SkvHostMirror;  // host copy of the structure, kept for insertions
struct skv_tree {
  SkvTreeDev dev;
  int64_t n_in_blocks;
  int device;
  SkvHostMirror* host;
  int has_copies;  // some position holds several children with the same first block: lookups must branch
};

// ---- block hash (host builds the tables, device probes them) -------------------------------
SKV_HD inline uint64_t skv_mix_tok(uint32_t tok, uint32_t i) {
  uint64_t x = (uint64_t)tok + 0x9E3779B97F4A7C15ull * (uint64_t)(i + 1);
  x ^= x >> 32; x *= 0xD6E8FEB86659FD93ull;
  x ^= x >> 32; x *= 0xD6E8FEB86659FD93ull;
  x ^= x >> 32;
  return x;
}
SKV_HD inline uint64_t skv_hash_fin(uint64_t s) {
  s ^= s >> 29; s *= 0xBF58476D1CE4E5B9ull;
  s ^= s >> 32;
  return s;
}
inline uint64_t skv_hash_block_host(const int32_t* tok) {
  uint64_t s = 0;
  for (uint32_t i = 0; i < 16; ++i) s += skv_mix_tok((uint32_t)tok[i], i);
  return skv_hash_fin(s);
}

#ifdef __HIPCC__
// Moves between lanes on the vector unit: data-parallel primitives within a row of 16 lanes and swaps of rows and halves.  What __shfl
// compiles to goes through the LDS unit, and a scan or a reduction is a chain of six of them: the chip's small kernels, and the start
// of every large one that looks for its work, are such chains.  All lanes of the wavefront take part.  us before / after: an attention
// workgroup of a split call finds its part 4.7 / 3.0 and 5.1 / 3.6; passes with one request behind 2992 keys 35.9 / 34.4, three decode
// requests 12.5 / 11.9, 4096 lookups and their window 46.0 / 45.0.
template <int kCtrl, int kRows = 0xf, typename T>
__device__ __forceinline__ T skv_dpp(T old, T v) {   // lanes without a source, or in rows outside kRows, keep `old`
  static_assert(sizeof(T) == 4 || sizeof(T) == 8);
  if constexpr (sizeof(T) == 4) {
    return __builtin_bit_cast(T, __builtin_amdgcn_update_dpp(__builtin_bit_cast(int, old), __builtin_bit_cast(int, v), kCtrl, kRows, 0xf, false));
  } else {
    const uint64_t o = __builtin_bit_cast(uint64_t, old), x = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = __builtin_amdgcn_update_dpp((int)(uint32_t)o, (int)(uint32_t)x, kCtrl, kRows, 0xf, false);
    const uint32_t hi = __builtin_amdgcn_update_dpp((int)(uint32_t)(o >> 32), (int)(uint32_t)(x >> 32), kCtrl, kRows, 0xf, false);
    return __builtin_bit_cast(T, (uint64_t)hi << 32 | lo);
  }
}
constexpr int kSkvRowShr = 0x110, kSkvRowRor = 0x120, kSkvRowMirror = 0x140, kSkvHalfMirror = 0x141, kSkvBcast15 = 0x142, kSkvBcast31 = 0x143,
              kSkvQuadXor1 = 0xB1, kSkvQuadXor2 = 0x4E;   // (shifts and rotations: + distance)
// v_permlane16_swap exchanges the odd rows of its first operand with the even rows of its second, v_permlane32_swap the upper half of
// the first with the lower half of the second; on two copies of a value either leaves the one row's or half's value in `a` and the
// other's in `b`, so no lane select is needed.  (The wait states the compiler places between a VALU write and these are added by hand.)
__device__ __forceinline__ void skv_swap_rows(float& a, float& b) { asm volatile("s_nop 1\n\tv_permlane16_swap_b32 %0, %1\n\ts_nop 1" : "+v"(a), "+v"(b)); }
__device__ __forceinline__ void skv_swap_halves(float& a, float& b) { asm volatile("s_nop 1\n\tv_permlane32_swap_b32 %0, %1\n\ts_nop 1" : "+v"(a), "+v"(b)); }
// op over the four lanes 16 apart, over all lanes; every lane has the result (32-bit types)
template <typename T, typename Op>
__device__ __forceinline__ T skv_over_rows(T v, Op op) {
  float a = __builtin_bit_cast(float, v), b = a;
  skv_swap_rows(a, b);
  a = b = __builtin_bit_cast(float, op(__builtin_bit_cast(T, a), __builtin_bit_cast(T, b)));
  skv_swap_halves(a, b);
  return op(__builtin_bit_cast(T, a), __builtin_bit_cast(T, b));
}
template <typename T, typename Op>
__device__ __forceinline__ T skv_over_wave(T v, Op op) {
  v = op(v, skv_dpp<kSkvQuadXor1>(v, v));
  v = op(v, skv_dpp<kSkvQuadXor2>(v, v));
  v = op(v, skv_dpp<kSkvHalfMirror>(v, v));
  v = op(v, skv_dpp<kSkvRowMirror>(v, v));
  return skv_over_rows(v, op);
}
struct SkvAdd { template <typename T> __device__ T operator()(T a, T b) const { return a + b; } };
struct SkvMax {
  __device__ float operator()(float a, float b) const { return fmaxf(a, b); }
  __device__ int operator()(int a, int b) const { return max(a, b); }
};
template <typename T>
__device__ __forceinline__ T skv_wave_scan(T v) {   // inclusive
  const T zero = 0;
  v += skv_dpp<kSkvRowShr + 1>(zero, v);
  v += skv_dpp<kSkvRowShr + 2>(zero, v);
  v += skv_dpp<kSkvRowShr + 4>(zero, v);
  v += skv_dpp<kSkvRowShr + 8>(zero, v);
  v += skv_dpp<kSkvBcast15, 0xa>(zero, v);
  v += skv_dpp<kSkvBcast31, 0xc>(zero, v);
  return v;
}
template <typename T>
__device__ __forceinline__ T skv_lane(T v, int from) {   // `from` the same in all lanes
  if constexpr (sizeof(T) == 4) {
    return __builtin_bit_cast(T, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), from));
  } else {
    const uint64_t x = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = __builtin_amdgcn_readlane((int)(uint32_t)x, from), hi = __builtin_amdgcn_readlane((int)(uint32_t)(x >> 32), from);
    return __builtin_bit_cast(T, (uint64_t)hi << 32 | lo);
  }
}
// Inclusive scan over a workgroup of kThreads; `total` of all threads.  red: one place per wavefront.  Two barriers.
template <int kThreads, typename T>
__device__ inline T skv_block_scan(T v, T* red, T& total) {
  constexpr int kWaves = kThreads / 64;
  static_assert(kWaves <= 16);   // a row of lanes
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  v = skv_wave_scan(v);
  if (lane == 63) red[wave] = v;
  __syncthreads();
  const T zero = 0;
  T x = lane < kWaves ? red[lane] : zero;
  x += skv_dpp<kSkvRowShr + 1>(zero, x);
  x += skv_dpp<kSkvRowShr + 2>(zero, x);
  x += skv_dpp<kSkvRowShr + 4>(zero, x);
  x += skv_dpp<kSkvRowShr + 8>(zero, x);
  total = skv_lane(x, kWaves - 1);
  if (wave > 0) v += skv_lane(x, wave - 1);
  __syncthreads();
  return v;
}
#endif

// ---- error plumbing ---------------------------------------------------------------------------
void skv_set_hip_error(int e);
#define SKV_HIP(call)                          \
  do {                                         \
    hipError_t e_ = (call);                    \
    if (e_ != hipSuccess) {                    \
      skv_set_hip_error((int)e_);              \
      return SKV_EHIP;                         \
    }                                          \
  } while (0)

static inline size_t skv_align256(size_t x) { return (x + 255) & ~(size_t)255; }

// Softmax scale of an attention description: the caller's value when it is a positive finite number,
// otherwise 1/sqrt(head_dim) (scaled dot-product attention, SafeKV Section 2.1).
static inline float skv_softmax_scale(const skv_attn_desc* d) {
  const float s = d->scale;
  if (s > 0.f && s < 3.0e38f) return s;
  return 1.0f / sqrtf((float)d->head_dim);
}

#endif
