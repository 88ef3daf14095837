// Causal GQA prefill attention of the uncached suffix over reused paged prefix KV plus the
// request's own new KV.
//
// SafeKV Section 2.1: inference attends over all previous tokens; with KV caching the K/V of
// the cached prefix are reused and only the new tokens' part is computed.  Row i of the
// suffix therefore attends to the L reused positions (read from the page pool through the
// page table the match produced) and to its own positions 0..i.
//
// bf16 path: flash-style streaming over 64-key tiles with online softmax in fp32; the two
// contractions (K.Q^T and V^T.P^T) run on the matrix cores (v_mfma_f32_32x32x16_bf16), the
// softmax on the vector ALU.  A workgroup of eight wavefronts shares every K/V tile through
// LDS; each wavefront owns 32 query rows of one head (the query heads of one kv head share a
// workgroup, so a K/V tile is fetched once for the group).  K/V rows travel global -> LDS with
// direct-to-LDS loads (no stop in registers, no LDS store instructions), three stages each.
// The products are formed transposed (S^T = K Q^T, O^T = V^T P^T) so that a query is a
// lane-column of the MFMA accumulator: row sums are register reductions, and the P^T
// accumulator registers are already in the B-operand layout of the second product; V^T
// fragments come from the LDS transpose load.  The inner loop is a three-stage software
// pipeline over 32-key sub-tiles: the scores of sub-tile h + 1, the softmax of sub-tile h and
// the output update with sub-tile h - 1 share a half-step, in which nothing depends on
// anything else, so MFMAs and vector instructions alternate in the instruction stream.
// fp32 path: skv_attn_f32.hip.
#include <atomic>

#include "skv_internal.h"

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

constexpr int kD = 128;          // head dim of the bf16 kernel
constexpr int kBN = 64;          // keys per LDS tile
constexpr int kKStages = 3;      // LDS stages of K: tiles kt, kt + 1 in use, kt + 2 arriving
constexpr int kVStages = 3;      // LDS stages of V: tiles kt - 1, kt in use, kt + 1 arriving
constexpr int kStageRows = 16;   // rows of a wave's Q / O staging tile
constexpr float kSumLimit = 4096.f;   // move the softmax reference when a lane's sum of 16 exponentials exceeds this
constexpr int kRowsPerWave = 32; // query rows per wavefront
constexpr int kWaves = 8;        // two per SIMD: one wave's softmax overlaps the other's MFMAs
constexpr int kThreads = kWaves * 64;
// LDS tile layout (K and V alike): a 64-key tile is 16 segments of 4 keys, 1040 bytes apart.  Inside a segment the
// 16-byte piece (key q of the segment, chunk c of the 256-byte row) sits at (c / 4) * 256 + q * 64 + (c % 4) * 16.
// One direct-to-LDS load of a wavefront fills one segment: the hardware puts what lane i fetched at byte 16 i, so
// lane i fetches chunk 4 (i / 16) + i % 4 of key (i / 4) % 4 -- four lanes read 64 consecutive bytes of a row.
// The K fragment reads (ds_read_b128: 16 lanes = 16 keys, one chunk) and the V^T fragment reads
// (ds_read_b64_tr_b16: 32 lanes = 4 keys x 64 bytes) are free of bank conflicts, and the addresses of different
// fragments differ by constants only.
constexpr int kSeg = 520;            // bf16 elements per segment (1040 B)
constexpr int kTile = 16 * kSeg;     // bf16 elements per 64-key tile
constexpr float kLog2e = 1.4426950408889634f;

struct AttnParams {
  const void *q, *knew, *vnew, *kpool, *vpool;
  void* out;
  const int32_t *q_off, *matched_len, *page_table;
  const int32_t* items;      // kItemInts ints per work item
  const int32_t* n_items;
  const char* zero_page;     // 16 rows of zeros: stands in for a group of keys that has no data
  const int32_t* splits;     // kSplitInts ints per work item whose keys are split over several workgroups
  float* partials;           // kSlotFloats floats per part and (kv head, head group); null: nothing is ever split
  int n_req, max_blocks, n_pages, Hq, Hkv;
  int heads_per_wg;          // query heads of one kv head handled by one workgroup (1, 2 or 4)
  float scale;
};

// ---- work list ---------------------------------------------------------------------------------
// One workgroup.  items[] lists one 32-byte record per (request, q tile) pair -- {request, first suffix row of
// the tile, first row of the request in Q, its suffix length S, its reused length L, end row of the tile, first key tile,
// part} -- so that a workgroup of the attention kernel learns everything about its piece of work from one load.  A request's
// heaviest (last) tile first.  The q tiles of a request are cut so that L + (first row of a tile) is a multiple of the
// 64-key tile: the first tile is short when L is not, and every later tile ends exactly where a key tile ends, so
// no workgroup streams a key tile for the sake of a few keys of round-up -- unless the short first tile makes the
// request one tile longer than cutting from row 0 would and the reused prefix is long (L > S / 2): a tile more costs
// a pass over about L + S / 2 keys, the round-up one more 64-key iteration in each of the S / 64 tiles.
//
// Small batches leave most of the chip idle and their time is the length of one workgroup's pass over the keys (one turn
// behind 24 k cached tokens: 80 workgroups, 0.50 ms).  Their items are split along the keys: every part is a record of its
// own (part = (slot + 1) << kPartBits | key tiles), leaves its unnormalised output, reference and row sum in the workspace,
// and attn_merge_kernel combines them.  The part length c is the smallest for which all parts run in one round, or in
// two, of one workgroup per compute unit; a workgroup costs about kStartTiles key tiles before and after its loop, the
// merge about as much again, and unless the split wins by that the items stay whole.
constexpr int kItemInts = 8;
constexpr int kCus = 256;             // compute units = workgroups that run at once
constexpr int kMaxSlots = 2 * kCus;   // parts of a split batch, over all kv heads and head groups
constexpr int kStartTiles = 8;
constexpr int kPartBits = 20;         // key tiles of a part
constexpr int kSplitInts = 8;         // {first row, end row, first row of the request in Q, first slot, parts, 0, 0, 0}
constexpr int kSlotFloats = kWaves * 64 * (64 + 2);   // per wavefront and lane: 64 of O^T, reference, row sum

struct Cut {   // how one request's suffix is cut into q tiles
  int S, L, qb, head_rows, nt;
  __device__ void tile(int j, int pos_per_wg, int& row0, int& row1) const {   // j-th tile from the front
    if (head_rows > 0 && j == 0) {
      row0 = 0;
      row1 = head_rows;
    } else {
      row0 = head_rows + (j - (head_rows > 0 ? 1 : 0)) * pos_per_wg;
      row1 = min(S, row0 + pos_per_wg);
    }
  }
};
__device__ inline Cut cut_of(int r, const int32_t* q_off, const int32_t* matched_len, int pos_per_wg) {
  Cut c;
  c.qb = q_off[r];
  c.S = q_off[r + 1] - c.qb;
  c.L = matched_len[r] > 0 ? matched_len[r] & ~(SKV_BLOCK_TOKENS - 1) : 0;   // whole blocks only
  c.head_rows = min(c.S, (kBN - c.L % kBN) % kBN);                           // rows of the short first tile (0: none)
  c.nt = c.S > 0 ? (c.head_rows > 0 ? 1 : 0) + (c.S - c.head_rows + pos_per_wg - 1) / pos_per_wg : 0;
  const int nt_plain = (c.S + pos_per_wg - 1) / pos_per_wg;
  if (nt_plain < c.nt && 2 * c.L > c.S) {   // the short first tile would cost a whole extra tile: cut from row 0 instead
    c.head_rows = 0;
    c.nt = nt_plain;
  }
  return c;
}
// Parts an item of n key tiles is split into at part length c: every part but the first starts at a key that all of the
// item's rows see (key tile `last` or before), so that each part has a finite row maximum from its first keys on.
__device__ inline int parts_of(int n, int last, int c) {
  int parts = (n + c - 1) / c;
  while (parts > 1 && (parts - 1) * ((n + parts - 1) / parts) > last) --parts;
  return parts;
}

constexpr int kSchedThreads = 1024;
__global__ __launch_bounds__(kSchedThreads) void attn_schedule_kernel(
    int n_req, const int32_t* __restrict__ q_off, const int32_t* __restrict__ matched_len, int pos_per_wg, int max_items,
    int units /* workgroups per item */, int32_t* __restrict__ n_items /* [0] items, [1] split items */,
    int32_t* __restrict__ items, int32_t* __restrict__ splits /* null: never split */, uint4* __restrict__ zero_page,
    int zero_vec) {
  __shared__ int32_t sh[kSchedThreads];
  __shared__ int32_t carry;
  for (int i = threadIdx.x; i < zero_vec; i += kSchedThreads) zero_page[i] = make_uint4(0u, 0u, 0u, 0u);
  if (threadIdx.x == 0) carry = 0;
  __syncthreads();
  for (int base = 0; base < n_req; base += kSchedThreads) {
    const int r = base + threadIdx.x;
    sh[threadIdx.x] = r < n_req ? cut_of(r, q_off, matched_len, pos_per_wg).nt : 0;
    __syncthreads();
    for (int o = 1; o < kSchedThreads; o <<= 1) {
      int add = threadIdx.x >= o ? sh[threadIdx.x - o] : 0;
      __syncthreads();
      sh[threadIdx.x] += add;
      __syncthreads();
    }
    // the chunk's items, one per thread and turn: the request is found in the scan
    const int first = carry, total = sh[kSchedThreads - 1];
    for (int it = threadIdx.x; it < total && first + it < max_items; it += kSchedThreads) {
      int lo = 0, hi = kSchedThreads - 1;   // smallest lo with sh[lo] > it
      while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (sh[mid] > it) hi = mid; else lo = mid + 1;
      }
      const Cut c = cut_of(base + lo, q_off, matched_len, pos_per_wg);
      int row0, row1;
      c.tile(sh[lo] - 1 - it, pos_per_wg, row0, row1);   // the request's last tile first
      int4* rec = (int4*)(items + (size_t)kItemInts * (first + it));
      rec[0] = make_int4(base + lo, row0, c.qb, c.S);
      rec[1] = make_int4(c.L, row1, 0, 0);
    }
    __syncthreads();
    if (threadIdx.x == 0) carry += total;
    __syncthreads();
  }
  const int n = min(carry, max_items);
  int n_out = n, n_split = 0;
  if (splits && n > 0 && n <= kCus && n * units <= kMaxSlots) {   // few items: split their keys?  One item per thread.
    __syncthreads();   // the records of the last chunk are read back below
    const int i = threadIdx.x;
    int4 a = {0, 0, 0, 0}, b = {0, 0, 0, 0};
    int n_kt = 0, last = 0;
    if (i < n) {
      a = ((const int4*)(items + (size_t)kItemInts * i))[0];
      b = ((const int4*)(items + (size_t)kItemInts * i))[1];
      n_kt = (b.x + b.y + kBN - 1) / kBN;
      last = (b.x + a.y) / kBN;
    }
    __shared__ int red[kCus / 64];
    auto block_sum = [&](int v) {   // over the first kCus threads
      for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o);
      if (i < kCus && (i & 63) == 0) red[i >> 6] = v;
      __syncthreads();
      int s = 0;
      for (int w = 0; w < kCus / 64; ++w) s += red[w];
      __syncthreads();
      return s;
    };
    int longest = n_kt;
    for (int o = 32; o >= 1; o >>= 1) longest = max(longest, __shfl_xor(longest, o));
    if (i < kCus && (i & 63) == 0) red[i >> 6] = longest;
    __syncthreads();
    longest = 0;
    for (int w = 0; w < kCus / 64; ++w) longest = max(longest, red[w]);
    __syncthreads();
    const int rounds_whole = (n * units + kCus - 1) / kCus;
    const int share = (block_sum(n_kt) * units + kCus - 1) / kCus;   // key tiles per compute unit
    const int whole = rounds_whole == 1 ? longest : max(longest, share + longest / 2);
    int best_c = longest, best_cost = rounds_whole * kStartTiles + whole - kStartTiles;   // (the split also merges)
    for (int rounds = 1; rounds <= 2; ++rounds) {
      const int room = rounds * kCus / units;
      if (room < n) continue;
      int lo = 1, hi = longest;   // smallest part length for which all parts have room
      while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (block_sum(i < n ? parts_of(n_kt, last, mid) : 0) <= room) hi = mid; else lo = mid + 1;
      }
      if (rounds * (kStartTiles + lo) < best_cost) {
        best_cost = rounds * (kStartTiles + lo);
        best_c = lo;
      }
    }
    const int parts = i < n ? parts_of(n_kt, last, best_c) : 0;
    const int total = block_sum(parts);
    if (total > n && total <= max_items) {
      // exclusive scans of the parts (place in the list), of the parts of split items (slot) and of the split items
      sh[i] = parts | (parts > 1 ? parts << 10 | 1 << 20 : 0);
      __syncthreads();
      for (int o = 1; o < kCus; o <<= 1) {
        const int add = i >= o && i < kCus ? sh[i - o] : 0;
        __syncthreads();
        if (i < kCus) sh[i] += add;
        __syncthreads();
      }
      if (i < n) {
        const int before = i ? sh[i - 1] : 0;
        const int at = before & 1023, slot = (before >> 10) & 1023, si = before >> 20;
        const int len = (n_kt + parts - 1) / parts;
        for (int j = 0; j < parts; ++j) {
          const int kt0 = j * len, n_part = min(len, n_kt - kt0);
          int4* rec = (int4*)(items + (size_t)kItemInts * (at + j));
          rec[0] = a;
          rec[1] = make_int4(b.x, b.y, kt0, parts > 1 ? (slot + j + 1) << kPartBits | n_part : 0);
        }
        if (parts > 1) {
          int4* sp = (int4*)(splits + kSplitInts * si);
          sp[0] = make_int4(a.y, b.y, a.z, slot);
          sp[1] = make_int4(parts, 0, 0, 0);
        }
      }
      n_out = total;
      n_split = sh[n - 1] >> 20;
    }
  }
  if (threadIdx.x == 0) {
    n_items[0] = n_out;
    n_items[1] = n_split;
  }
}

// ---- bf16 MFMA kernel --------------------------------------------------------------------------
// Value of the lane 32 positions away (the other half of the wavefront): v_permlane32_swap exchanges the
// upper half of its first operand with the lower half of its second.
__device__ inline float swap_halves(float x) {
  float a = x, b = x;
  // the wait states the compiler places between a VALU write and this instruction are added by hand
  asm volatile("s_nop 1\n\tv_permlane32_swap_b32 %0, %1\n\ts_nop 1" : "+v"(a), "+v"(b));
  return (threadIdx.x & 32) ? a : b;
}
// max / sum of a value and the one 32 lanes away: after the swap `a` holds the lower half's value in both halves
// and `b` the upper half's, so no lane select is needed
__device__ inline float max_halves(float x) {
  float a = x, b = x;
  asm volatile("s_nop 1\n\tv_permlane32_swap_b32 %0, %1\n\ts_nop 1" : "+v"(a), "+v"(b));
  return fmaxf(a, b);
}

// LDS fragment reads as inline assembly, with their waits placed by hand.  The compiler puts a full
// s_waitcnt vmcnt(0) in front of LDS reads it cannot tell apart from the targets of the direct-to-LDS loads in
// flight, which would stall every tile on the copies of the next one; the tile barrier already orders those
// copies against the reads.  The LDS returns data in issue order, so "at most n operations outstanding" means that
// everything issued before the n youngest reads has arrived.  A wait takes the registers it guards as in/out
// operands: their consumers then depend on it and cannot be moved in front of it.
__device__ __forceinline__ uint32_t lds_addr(const void* ptr) {
  return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const void*)ptr;
}
__device__ __forceinline__ bf16x8 lds_read_b128(uint32_t addr, int byte_off) {
  bf16x8 v;
  asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "i"(byte_off));
  return v;
}
__device__ __forceinline__ s16x4 lds_read_tr16_b64(uint32_t addr, int byte_off) {
  s16x4 v;
  asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "i"(byte_off));
  return v;
}
__device__ __forceinline__ void lds_wait(int n, bf16x8& a) {
  asm volatile("s_waitcnt lgkmcnt(%1)" : "+v"(a) : "i"(n));
}
__device__ __forceinline__ void lds_wait(int n, bf16x8& a, bf16x8& b, bf16x8& c, bf16x8& d) {
  asm volatile("s_waitcnt lgkmcnt(%4)" : "+v"(a), "+v"(b), "+v"(c), "+v"(d) : "i"(n));
}

__global__ __launch_bounds__(kThreads, 2) void attn_bf16_kernel(AttnParams p) {
  __shared__ __attribute__((aligned(16))) __bf16 smem[kKStages * kTile + kVStages * kTile +
                                                      kWaves * kStageRows * kD];
  __bf16* const Ks = smem;
  __bf16* const Vs = smem + kKStages * kTile;
  // [kWaves][16 rows][16 chunks of 8 bf16]: each wave's own staging tile for its Q rows on the way in and its O rows
  // on the way out (16 rows at a time), 16-byte chunks XOR-swizzled by row so that row-wise and fragment-wise
  // accesses are conflict free
  __bf16* const stage = Vs + kVStages * kTile + (threadIdx.x >> 6) * (kStageRows * kD);

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform by construction
  const int l32 = lane & 31;
  const int half = lane >> 5;

  // ---- which piece of work: XCD-aware decode (workgroup b runs on XCD b % 8) ----
  const int G = p.Hq / p.Hkv;
  const int n_hg = G / p.heads_per_wg;               // head groups per kv head
  int item, kvh, hg;
  {
    const int b = blockIdx.x;
    if (p.Hkv % 8 == 0) {
      // all work of one kv head stays on one XCD, so its K/V tiles are re-read from that XCD's L2
      const int per = p.Hkv / 8;
      const int xcd = b & 7, slot = b >> 3;
      kvh = xcd + 8 * (slot % per);
      const int rest = slot / per;
      hg = rest % n_hg;
      item = rest / n_hg;
    } else {
      kvh = b % p.Hkv;
      const int rest = b / p.Hkv;
      hg = rest % n_hg;
      item = rest / n_hg;
    }
  }
  // the record is read together with the item count (the grid bound keeps the index inside the list)
  const int4 rec0 = ((const int4*)(p.items + (size_t)kItemInts * item))[0];
  const int4 rec1 = ((const int4*)(p.items + (size_t)kItemInts * item))[1];
  if (item >= *p.n_items) return;
  const int kt0 = __builtin_amdgcn_readfirstlane(rec1.z);    // first key tile of this part
  const int part = __builtin_amdgcn_readfirstlane(rec1.w);   // 0: the whole item
  // Everything below counts keys from the part's first one: the reused length and with it every position shifts.
  const int L = __builtin_amdgcn_readfirstlane(rec1.x) - kt0 * kBN;                         // may be negative
  const int row1 = __builtin_amdgcn_readfirstlane(rec1.y);                                  // end row of the q tile
  const int r = __builtin_amdgcn_readfirstlane(rec0.x);
  const int row0 = __builtin_amdgcn_readfirstlane(rec0.y);                                  // first row of the q tile
  const int qbase = __builtin_amdgcn_readfirstlane(rec0.z);
  const int S = __builtin_amdgcn_readfirstlane(rec0.w);
  const int Ltot = L + S;

  const int head = kvh * G + hg * p.heads_per_wg + (wave % p.heads_per_wg);
  const int pos0 = row0 + (wave / p.heads_per_wg) * kRowsPerWave;             // first row of this wave
  const int n_tiles = part ? part & ((1 << kPartBits) - 1) : (L + row1 + kBN - 1) / kBN;   // 64-key tiles the workgroup streams
  const int wave_key_end = pos0 < row1 ? min(L + min(row1, pos0 + kRowsPerWave), n_tiles * kBN) : 0;  // this wave needs keys [0, wave_key_end)
  const int32_t* const table = p.page_table + (size_t)r * p.max_blocks + kt0 * (kBN / SKV_BLOCK_TOKENS);
  const int table_len = p.max_blocks - kt0 * (kBN / SKV_BLOCK_TOKENS);

  // ---- the first global reads, all in flight together: the page ids of the first two address windows (what the K/V
  // loads need first), then this wave's Q rows.  The K/V loads are issued as soon as the page ids are there; Q is
  // staged while they travel.
  // A window is fetched in two parts, so that the page-table read can be in flight while other work goes on: the
  // page id first, the addresses from it later.
  auto window_page = [&](int w) __attribute__((always_inline)) {
    const int gi = w * 64 + lane;
    int page = -1;
    if (gi * SKV_BLOCK_TOKENS < L && gi < table_len) page = __builtin_nontemporal_load(&table[gi]);
    return page;
  };
  // (the five base addresses as values: selecting between the fields of the argument block itself makes the
  // compiler select their addresses and load through them, a vector-memory read that everything behind it waits for)
  const uint64_t kpool_a = (uint64_t)p.kpool, vpool_a = (uint64_t)p.vpool, knew_a = (uint64_t)p.knew,
                 vnew_a = (uint64_t)p.vnew, zero_a = (uint64_t)p.zero_page;
  auto window_bases = [&](int w, int page, uint64_t& ak, uint64_t& av) __attribute__((always_inline)) {
    const int gi = w * 64 + lane;
    const int key0 = gi * SKV_BLOCK_TOKENS;
    uint64_t k = zero_a, v = zero_a;
    if (key0 < L) {
      if (page >= 0 && page < p.n_pages) {
        const uint64_t off = ((uint64_t)page * SKV_BLOCK_TOKENS * p.Hkv + kvh) * (kD * 2);
        k = kpool_a + off;
        v = vpool_a + off;
      }
    } else if (key0 < Ltot) {
      const uint64_t off = ((uint64_t)(qbase + key0 - L) * p.Hkv + kvh) * (kD * 2);
      k = knew_a + off;
      v = vnew_a + off;
    }
    ak = k;
    av = v;
  };
  const int page_w0 = window_page(0), page_w1 = window_page(1);

  // ---- Q fragments (B operand of S^T = K Q^T): lane holds query l32, d = 16 ks + 8 half .. +7
  // Rows are fetched whole (16 lanes x 16 B per row) and picked up from the wave's staging tile.  The scores leave the
  // matrix core unscaled; scale * log2(e) is applied in fp32 by the multiply-add that also subtracts the reference
  // (scaling Q itself would round it to bf16 a second time: visible when scores spread over hundreds of units).
  const float c = p.scale * kLog2e;
  bf16x8 qf[8];
  u32x4 qv[8];
  {
    const int c16 = lane & 15;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int rr = (lane >> 4) + 4 * i;
      const int row = min(pos0 + rr, S - 1);   // rows past the tile or the request are computed and dropped
      qv[i] = *(const u32x4*)((const __bf16*)p.q + ((size_t)(qbase + row) * p.Hq + head) * kD + c16 * 8);
    }
  }
  auto stage_q = [&]() __attribute__((always_inline)) {
    const int c16 = lane & 15;
#pragma unroll
    for (int pass = 0; pass < 2; ++pass) {   // the staging tile takes 16 rows at a time
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int rr = (lane >> 4) + 4 * i;    // row within the pass
        *(u32x4*)(stage + rr * kD + ((c16 ^ rr) << 3)) = qv[4 * pass + i];
      }
      if ((l32 >> 4) == pass) {
        const int rr = l32 & 15;
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) qf[ks] = *(const bf16x8*)(stage + rr * kD + (((2 * ks + half) ^ rr) << 3));
      }
    }
  };

  f32x16 o[4];   // O^T accumulators: d = 32 a + 8(e/4) + 4 half + e%4, query = l32
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int e = 0; e < 16; ++e) o[a][e] = 0.f;

  // ---- global -> LDS, without a stop in registers ----
  // A tile is four 16-key groups; a group is one page of the pool or 16 consecutive new rows.  Each wavefront
  // moves two segments of a tile (segments w and w + 8: keys 4w.. and 32 + 4w..) with direct-to-LDS loads: lane i
  // fetches chunk 4 (i / 16) + i % 4 of key (i / 4) % 4 of the segment and the hardware puts it at slot i.
  const unsigned row_bytes = (unsigned)p.Hkv * kD * 2u;
  const int t_row = (wave & 3) * 4 + ((lane >> 2) & 3);      // row of the 16-key group this lane fetches
  const unsigned t_col = (unsigned)((lane >> 4) * 4 + (lane & 3)) * 16u;
  const unsigned t_off = (unsigned)t_row * row_bytes + t_col;
  // Group base addresses, one 16-key group per lane for 64 groups (16 tiles, a "window"): a pool page, 16 new rows,
  // or the page of zeros when the group has no data (past the end of the sequence, or a page id outside the pool).
  // A tile's bases are read with lane broadcasts.  Two consecutive windows are held; K tiles run one tile ahead of
  // V tiles, so for one iteration in sixteen K reads the later window while V still reads the earlier one.
  auto lane_bcast = [&](uint64_t x, int idx) __attribute__((always_inline)) {
    const uint32_t lo = __builtin_amdgcn_readlane((int)(uint32_t)x, idx);
    const uint32_t hi = __builtin_amdgcn_readlane((int)(uint32_t)(x >> 32), idx);
    return (const __attribute__((address_space(1))) char*)(((uint64_t)hi << 32) | lo);   // global, not flat
  };
  uint64_t ak_cur, av_cur, ak_nxt, av_nxt;
  int win = 0;                       // window held in *_cur; *_nxt holds window win + 1
  window_bases(0, page_w0, ak_cur, av_cur);
  window_bases(1, page_w1, ak_nxt, av_nxt);
  typedef __attribute__((address_space(3))) void lds_void;
  // one pool (K or V) of tile t into an LDS stage; `bases` holds the window of tile t
  auto load_half_tile = [&](uint64_t bases, int t, __bf16* dst_stage) __attribute__((always_inline)) {
    const int key_base = t * kBN;
    __bf16* const dst = dst_stage + wave * kSeg;
#pragma unroll
    for (int cc = 0; cc < 2; ++cc) {
      const int g = (wave >> 2) + 2 * cc;                    // 16-key group of segment wave + 8 cc
      const int idx = ((t & 15) << 2) + g;
      const auto gb = lane_bcast(bases, idx);
      unsigned off = t_off;
      if (key_base + kBN > Ltot) {  // the sequence ends inside this tile: rows past its end re-read its last row,
        const int n_valid = Ltot - (key_base + g * 16);  // finite values that the causal mask keeps out
        if (n_valid > 0 && n_valid < 16) off = (unsigned)min(t_row, n_valid - 1) * row_bytes + t_col;
      }
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(gb + off),
                                       (lds_void*)(dst + cc * 8 * kSeg), 16, 0, 0);
    }
  };
  auto load_k_tile = [&](int t, int stage_idx) __attribute__((always_inline)) {
    load_half_tile((t >> 4) == win ? ak_cur : ak_nxt, t, Ks + stage_idx * kTile);
  };
  auto load_v_tile = [&](int t, int stage_idx) __attribute__((always_inline)) {
    load_half_tile((t >> 4) == win ? av_cur : av_nxt, t, Vs + stage_idx * kTile);
  };
  // Inside the main loop the same loads are split in two: the segment bases of the tiles an iteration will request
  // (K two tiles ahead, V one) are broadcast out of the windows during the iteration before, between its half-steps,
  // so that the iteration itself starts with nothing but the four load instructions.  Right after a barrier every
  // wave of the workgroup is at this point at once, and what stands here keeps all matrix cores waiting.
  typedef const __attribute__((address_space(1))) char* gptr;
  gptr nk[2], nv[2];
  int pend_page = -1;
  bool pend = false;
  auto prep_bases = [&](int kt_next) __attribute__((always_inline)) {
    if (((kt_next + 1) >> 4) != win) {   // V enters the next window: move on and ask for the page ids of the one
      ++win;                             // after it; K needs that window fourteen iterations from now, the iteration
      ak_cur = ak_nxt;                   // after this one turns the ids into addresses, behind its barrier, where
      av_cur = av_nxt;                   // every load of this wave has landed anyway
      pend_page = window_page(win + 1);
      pend = true;
    }
    const int tk = kt_next + 2, tv = kt_next + 1;
#pragma unroll
    for (int cc = 0; cc < 2; ++cc) {
      const int g = (wave >> 2) + 2 * cc;
      nk[cc] = lane_bcast((tk >> 4) == win ? ak_cur : ak_nxt, ((tk & 15) << 2) + g);
      nv[cc] = lane_bcast((tv >> 4) == win ? av_cur : av_nxt, ((tv & 15) << 2) + g);
    }
  };
  auto issue_half_tile = [&]<bool kWhole>(const gptr (&b)[2], int t, __bf16* dst_stage) __attribute__((always_inline)) {
    const int key_base = t * kBN;
    __bf16* const dst = dst_stage + wave * kSeg;
#pragma unroll
    for (int cc = 0; cc < 2; ++cc) {
      unsigned off = t_off;
      if (!kWhole && key_base + kBN > Ltot) {   // as in load_half_tile
        const int n_valid = Ltot - (key_base + ((wave >> 2) + 2 * cc) * 16);
        if (n_valid > 0 && n_valid < 16) off = (unsigned)min(t_row, n_valid - 1) * row_bytes + t_col;
      }
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(b[cc] + off),
                                       (lds_void*)(dst + cc * 8 * kSeg), 16, 0, 0);
    }
  };
  // a wave's direct loads are in LDS once its vector-memory counter has drained; the barrier then publishes them
  auto tile_barrier = [&]() __attribute__((always_inline)) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
  };

  // ---- the steps of the pipeline ----
  // Work advances in 32-key sub-tiles (half an LDS tile), three of them in flight: half-step h puts the scores of
  // sub-tile h + 1 and the output update with sub-tile h - 1 on the matrix core and computes the softmax of sub-tile
  // h on the vector ALU.  Nothing inside a half-step depends on anything else inside it, so its 16 MFMAs alternate
  // (score, output, score, ...) with two or three vector instructions behind each: the vector work runs beside the
  // MFMAs instead of between them.  Two score accumulators and two P^T buffers alternate.
  f32x16 s[2];      // S^T of two consecutive sub-tiles: [32 keys][32 queries], raw dot products
  bf16x8 pb[2][2];  // P^T as B operands: [sub-tile parity][16-key group]
  bf16x8 kfr[4];    // K fragment ring: runs four fragments ahead, across sub-tiles
  bf16x8 vfr[4];    // V^T fragment ring, likewise
  float m_ref = 0.f;   // reference the exponentials are taken against (score * scale * log2(e): exp2 units), per query
  float l_run = 0.f;   // running row sum over this lane-half's keys
#pragma unroll
  for (int e = 0; e < 16; ++e) s[0][e] = s[1][e] = 0.f;
  const f32x16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int e = 0; e < 8; ++e) pb[0][0][e] = pb[0][1][e] = pb[1][0][e] = pb[1][1][e] = (__bf16)0.f;
  // K fragment (ks, mt): lane (l32, half) wants key l32 + 32 mt, chunk 2 ks + half.  In bf16 elements:
  //   segment (l32 / 4 + 8 mt) * kSeg + key-in-segment (l32 % 4) * 32 + (ks / 2) * 128 + (2 (ks % 2) + half) * 8
  const int k_lane = (l32 >> 2) * kSeg + (l32 & 3) * 32 + half * 8;
  // The PV A operand wants, per lane (d = 32 a + l32), the eight keys {4 half + 0..3, 8 + 4 half + 0..3}
  // of a 16-key group -- the keys this lane-half's P^T registers hold.  Each quad comes from one LDS
  // transpose load: within 16 lanes, lane i supplies the address of 4 consecutive d of key (i / 4) at d
  // offset 4 (i % 4) and receives d offset i of the four keys.  For fragment (g16, a) the lane's key is
  // 16 g16 + 4 half + (lane % 16) / 4 (segment 4 g16 + half, second load two segments on) and its 8 bytes are piece
  // lane % 2 of chunk 4 a + 2 ((lane / 16) % 2) + (lane % 4) / 2.
  const int v_lane = half * kSeg + ((lane & 15) >> 2) * 32 + (2 * ((lane >> 4) & 1) + ((lane & 3) >> 1)) * 8 + 4 * (lane & 1);
  // fragment addresses are LDS byte addresses: a per-lane base plus constants that fit the offset field
  auto k_frag = [&](uint32_t kb, int ks) __attribute__((always_inline)) {   // kb: stage + k_lane + mt * 8 kSeg
    return lds_read_b128(kb, ((ks >> 1) * 128 + (ks & 1) * 16) * 2);
  };
  auto v_frag = [&](uint32_t vb, int j) __attribute__((always_inline)) {   // vb: stage + v_lane + h * 8 kSeg; j = (g, a)
    const int off = ((j >> 2) * 4 * kSeg + (j & 3) * 128) * 2;
    const s16x4 lo = lds_read_tr16_b64(vb, off);
    const s16x4 hi = lds_read_tr16_b64(vb, off + 2 * kSeg * 2);
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
  };
  // causal mask of sub-tile u (keys 32 u ..), applied where the sub-tile reaches past the wave's first row
  auto mask = [&](f32x16& x, int u) __attribute__((always_inline)) {
    const int key0 = u * 32;
    if (key0 + 31 > L + pos0) {
      const int limit = L + pos0 + l32;  // last visible key of this lane's query
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int key = key0 + (e >> 2) * 8 + half * 4 + (e & 3);
        if (key > limit) x[e] = -INFINITY;
      }
    }
  };
  auto row_max = [&](const f32x16& x) __attribute__((always_inline)) {
    float m4[4];   // four independent reduction chains
#pragma unroll
    for (int k = 0; k < 4; ++k) m4[k] = fmaxf(x[k], x[k + 4]);
#pragma unroll
    for (int e = 8; e < 16; ++e) m4[e & 3] = fmaxf(m4[e & 3], x[e]);
    float mx = fmaxf(fmaxf(m4[0], m4[1]), fmaxf(m4[2], m4[3]));
    return max_halves(mx);
  };
  // exponentials of one pair of scores -> packed bf16, plain fp32 adds for the row sum (the packed dot-product
  // instruction that would add the pair in one step does not run beside the MFMAs, the adds do)
  float ssum[2];
  bf16x8 pk;
  auto exp_pair = [&](const f32x16& cur, int i, bf16x8 (&p_make)[2], float& e0, float& e1, int part) __attribute__((always_inline)) {
    if (part == 0) {
      e0 = __builtin_amdgcn_exp2f(__builtin_fmaf(cur[2 * i], c, -m_ref));
      e1 = __builtin_amdgcn_exp2f(__builtin_fmaf(cur[2 * i + 1], c, -m_ref));
    } else {
      f32x2 pr = {e0, e1};
      const bf16x2 cv = __builtin_convertvector(pr, bf16x2);
      ssum[0] += e0;
      ssum[1] += e1;
      pk[2 * (i & 3)] = cv[0];
      pk[2 * (i & 3) + 1] = cv[1];
      if ((i & 3) == 3) p_make[i >> 2] = pk;
    }
  };
  // The softmax keeps a reference per query; exponentials are taken against it as it stands, which leaves the
  // normalised result unchanged.  Only when a lane's sum of exponentials over a sub-tile passes kSumLimit (an element
  // at least kSumLimit / 16 above the reference; infinities and NaNs trip it too) is the reference moved to that
  // sub-tile's row maximum: O and the row sum are rescaled and this sub-tile's exponentials are taken again.  This
  // happens between half-steps, after the output update that still belongs to the old reference has been issued.
  auto move_reference = [&](const f32x16& cur, bf16x8 (&p_make)[2]) __attribute__((always_inline)) {
    const float mx = row_max(cur) * c;
    const bool trip = !(max_halves(ssum[0] + ssum[1]) <= kSumLimit);
    const float m_new = trip ? mx : m_ref;
    const float alpha = __builtin_amdgcn_exp2f(m_ref - m_new);
    m_ref = m_new;
    l_run *= alpha;
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int e = 0; e < 16; ++e) o[a][e] *= alpha;
    ssum[0] = ssum[1] = 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      float e0, e1;
      exp_pair(cur, i, p_make, e0, e1, 0);
      exp_pair(cur, i, p_make, e0, e1, 1);
    }
  };
  auto active = [&](int u) __attribute__((always_inline)) { return u * 32 < wave_key_end; };
  // One half-step.  kb / kb_next: K of sub-tiles h + 1 and h + 2; vb / vb_next: V of sub-tiles h - 1 and h.
  // The rings hold fragments 0..3 of sub-tile h + 1 (K) and of sub-tile h - 1 (V^T) on entry and are refilled behind
  // each MFMA with fragments 4..7 and then with fragments 0..3 of the following sub-tile.
  // Fast form (every stage at work, no masked key in sub-tile h): the 16 MFMAs alternate and carry the softmax between
  // them; a fragment is waited for four pair-steps after its request, with eleven (K) or ten (V^T) younger reads.
  auto half_step_fast = [&]<bool kMask>(int h, uint32_t kb, uint32_t kb_next, uint32_t vb, uint32_t vb_next, f32x16& dst,
                                        f32x16& cur, bf16x8 (&p_use)[2], bf16x8 (&p_make)[2]) __attribute__((always_inline)) {
    if (kMask) mask(cur, h);
    ssum[0] = ssum[1] = 0.f;
    // One exponential behind every MFMA, never two in a row: the transcendental unit takes about four issue slots
    // per instruction but works beside the issue port, so a second one right behind the first would hold the
    // wavefront until the unit is free again.  The pair is packed and summed one step later, behind the next
    // exponential.
    float e0 = 0.f, e1 = 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      lds_wait(11, kfr[i & 3]);
      dst = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kfr[i & 3], qf[i], i == 0 ? zero16 : dst, 0, 0, 0);
      kfr[i & 3] = i < 4 ? k_frag(kb, i + 4) : k_frag(kb_next, i - 4);
      const float f0 = __builtin_amdgcn_exp2f(__builtin_fmaf(cur[2 * i], c, -m_ref));
      if (i > 0) {
        f32x2 pr = {e0, e1};
        const bf16x2 cv = __builtin_convertvector(pr, bf16x2);
        pk[2 * ((i - 1) & 3)] = cv[0];
        pk[2 * ((i - 1) & 3) + 1] = cv[1];
        ssum[0] += e0;
      }
      __builtin_amdgcn_sched_barrier(0);
      lds_wait(10, vfr[i & 3]);
      o[i & 3] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vfr[i & 3], p_use[i >> 2], o[i & 3], 0, 0, 0);
      vfr[i & 3] = i < 4 ? v_frag(vb, i + 4) : v_frag(vb_next, i - 4);
      const float f1 = __builtin_amdgcn_exp2f(__builtin_fmaf(cur[2 * i + 1], c, -m_ref));
      if (i > 0) {
        ssum[1] += e1;
        if (((i - 1) & 3) == 3) p_make[(i - 1) >> 2] = pk;
      }
      e0 = f0;
      e1 = f1;
      __builtin_amdgcn_sched_barrier(0);
    }
    {
      f32x2 pr = {e0, e1};
      const bf16x2 cv = __builtin_convertvector(pr, bf16x2);
      pk[6] = cv[0];
      pk[7] = cv[1];
      ssum[0] += e0;
      ssum[1] += e1;
      p_make[1] = pk;
    }
    if (__builtin_expect(__any(!(ssum[0] + ssum[1] <= kSumLimit)), 0)) move_reference(cur, p_make);
    l_run += ssum[0] + ssum[1];
  };
  // General form (first and last iterations of a wave): each stage is tested, runs as a block of its own, and waits
  // for every outstanding read.
  auto half_step_slow = [&](int h, uint32_t kb, uint32_t kb_next, uint32_t vb, uint32_t vb_next, f32x16& dst,
                            f32x16& cur, bf16x8 (&p_use)[2], bf16x8 (&p_make)[2]) __attribute__((always_inline)) {
    if (active(h + 1)) {
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        lds_wait(0, kfr[i & 3]);
        dst = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kfr[i & 3], qf[i], i == 0 ? zero16 : dst, 0, 0, 0);
        kfr[i & 3] = i < 4 ? k_frag(kb, i + 4) : k_frag(kb_next, i - 4);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    if (h > 0 && active(h - 1)) {
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        lds_wait(0, vfr[i & 3]);
        o[i & 3] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vfr[i & 3], p_use[i >> 2], o[i & 3], 0, 0, 0);
        vfr[i & 3] = i < 4 ? v_frag(vb, i + 4) : v_frag(vb_next, i - 4);
        __builtin_amdgcn_sched_barrier(0);
      }
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j) vfr[j] = v_frag(vb_next, j);   // the ring enters the next half-step as it expects
      __builtin_amdgcn_sched_barrier(0);
    }
    if (active(h)) {
      mask(cur, h);
      ssum[0] = ssum[1] = 0.f;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        float e0, e1;
        exp_pair(cur, i, p_make, e0, e1, 0);
        exp_pair(cur, i, p_make, e0, e1, 1);
      }
      if (__builtin_expect(__any(!(ssum[0] + ssum[1] <= kSumLimit)), 0)) move_reference(cur, p_make);
      l_run += ssum[0] + ssum[1];
    }
    // whatever follows finds every fragment of the rings in place
    lds_wait(0, kfr[0], kfr[1], kfr[2], kfr[3]);
    lds_wait(0, vfr[0], vfr[1], vfr[2], vfr[3]);
  };

  // ---- prologue: tiles K(0), K(1), V(0); scores of sub-tile 0; the reference starts at its row maxima
  load_k_tile(0, 0);
  if (n_tiles > 1) load_k_tile(1, 1);
  load_v_tile(0, 0);
  stage_q();
  tile_barrier();
  const uint32_t k_base = lds_addr(Ks + k_lane), v_base = lds_addr(Vs + v_lane);
  constexpr uint32_t kStageBytes = kTile * 2, kHalfBytes = 8 * kSeg * 2;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    kfr[j] = k_frag(k_base, j);
    vfr[j] = kfr[j];   // defined; the V^T ring fills itself during half-step 0
  }
  if (active(0)) {
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) {
      lds_wait(0, kfr[ks & 3]);
      s[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kfr[ks & 3], qf[ks], ks == 0 ? zero16 : s[0], 0, 0, 0);
      kfr[ks & 3] = ks < 4 ? k_frag(k_base, ks + 4) : k_frag(k_base + kHalfBytes, ks - 4);
      __builtin_amdgcn_sched_barrier(0);
    }
    // (idle states for the last MFMA: the compiler's wait-state insertion does not look through the branch inside
    // mask(), and the row maximum behind it would read score registers the matrix core has not written yet)
    asm volatile("s_nop 7\n\ts_nop 7\n\ts_nop 3" : "+v"(s[0]));
    mask(s[0], 0);
    m_ref = row_max(s[0]) * c;   // finite: key 0 is visible to every query
  }

  // ---- main loop.  Iteration kt (two half-steps) reads K(kt), K(kt + 1), V(kt - 1), V(kt).  It starts behind the
  // barrier that published K(kt + 1) and V(kt) and behind which no wave still reads K(kt - 1) or V(kt - 2): their
  // stages take the direct loads of K(kt + 2) and V(kt + 1), in flight during the whole iteration.  One barrier per
  // tile; one more iteration than tiles, for the output update with the last sub-tile.
  // Iterations [1, kt_fast) of this wave have all three stages at work, no masked key and no ragged tile to load.
  const int kt_fast = min(min((L + pos0 - 63) / 64 + 1, (wave_key_end - 1) / 64), n_tiles - 3);
  // Iterations [kt_fast, kt_mid) still have all three stages at work in both half-steps, but keys may be masked and
  // the tiles they request may be ragged or absent (the last two or three before the diagonal tile): they run the
  // fast form with the mask applied and the general loads.
  const int kt_mid = (wave_key_end - 1) / 64;
  int st0 = 0;   // stage of K(kt) and V(kt); tile t sits in stage t % 3
  auto iteration = [&]<int kForm>(int kt) __attribute__((always_inline)) {   // 0 general, 1 fast, 2 fast with masks
    constexpr bool kFast = kForm == 1;
    const int st1 = st0 == 2 ? 0 : st0 + 1;    // stage of tile kt + 1
    const int st2 = st1 == 2 ? 0 : st1 + 1;    // stage of tiles kt + 2 and kt - 1
    if (__builtin_expect(pend, 0)) {
      window_bases(win + 1, pend_page, ak_nxt, av_nxt);
      pend = false;
    }
    if (kFast || kt + 2 < n_tiles) issue_half_tile.template operator()<kFast>(nk, kt + 2, Ks + st2 * kTile);
    if (kFast || kt + 1 < n_tiles) issue_half_tile.template operator()<kFast>(nv, kt + 1, Vs + st1 * kTile);
    const uint32_t kb0 = k_base + st0 * kStageBytes;   // K(kt)
    const uint32_t kb1 = k_base + st1 * kStageBytes;   // K(kt + 1)
    const uint32_t vbp = v_base + st2 * kStageBytes;   // V(kt - 1)
    const uint32_t vb0 = v_base + st0 * kStageBytes;   // V(kt)
    if (kForm == 1) {
      half_step_fast.template operator()<false>(2 * kt, kb0 + kHalfBytes, kb1, vbp + kHalfBytes, vb0, s[1], s[0], pb[1], pb[0]);
      prep_bases(kt + 1);
      half_step_fast.template operator()<false>(2 * kt + 1, kb1, kb1 + kHalfBytes, vb0, vb0 + kHalfBytes, s[0], s[1], pb[0], pb[1]);
    } else if (kForm == 2) {
      half_step_fast.template operator()<true>(2 * kt, kb0 + kHalfBytes, kb1, vbp + kHalfBytes, vb0, s[1], s[0], pb[1], pb[0]);
      prep_bases(kt + 1);
      half_step_fast.template operator()<true>(2 * kt + 1, kb1, kb1 + kHalfBytes, vb0, vb0 + kHalfBytes, s[0], s[1], pb[0], pb[1]);
    } else {
      half_step_slow(2 * kt, kb0 + kHalfBytes, kb1, vbp + kHalfBytes, vb0, s[1], s[0], pb[1], pb[0]);
      prep_bases(kt + 1);
      half_step_slow(2 * kt + 1, kb1, kb1 + kHalfBytes, vb0, vb0 + kHalfBytes, s[0], s[1], pb[0], pb[1]);
    }
    tile_barrier();
    st0 = st1;
  };
  int kt = 0;
  prep_bases(0);
  iteration.template operator()<0>(kt++);
  for (; kt < kt_fast; ++kt) iteration.template operator()<1>(kt);
  for (; kt < kt_mid; ++kt) iteration.template operator()<2>(kt);
  for (; kt <= n_tiles; ++kt) iteration.template operator()<0>(kt);

  // ---- a part of a split item: O^T as it lies in the registers, the reference and the row sum
  if (pos0 >= row1) return;
  if (part) {
    const int slot = (part >> kPartBits) - 1;
    const int unit = kvh * n_hg + hg;
    f32x4* dst = (f32x4*)(p.partials + ((size_t)slot * p.Hkv * n_hg + unit) * kSlotFloats + (size_t)wave * (64 * 66)) + lane;
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int i4 = 0; i4 < 4; ++i4)
        dst[(a * 4 + i4) * 64] = f32x4{o[a][i4 * 4], o[a][i4 * 4 + 1], o[a][i4 * 4 + 2], o[a][i4 * 4 + 3]};
    float* ml = (float*)(dst - lane + 16 * 64) + lane;
    ml[0] = m_ref;
    ml[64] = l_run + swap_halves(l_run);
    return;
  }

  // ---- normalise and store.  A lane holds query l32 with d = 32 a + 8 (e/4) + 4 half + e%4, i.e. sixteen 8-byte
  // pieces of one output row.  They go through the wave's staging tile, 16 rows at a time, and leave as whole
  // 256-byte rows.
  {
    const float lsum = l_run + swap_halves(l_run);
    const float inv = 1.0f / lsum;
    const int c16 = lane & 15;
#pragma unroll
    for (int pass = 0; pass < 2; ++pass) {
      if ((l32 >> 4) == pass) {
        const int rr = l32 & 15;
        __bf16* row = stage + rr * kD;
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
          for (int i4 = 0; i4 < 4; ++i4) {
            f32x2 x0 = {o[a][i4 * 4 + 0] * inv, o[a][i4 * 4 + 1] * inv};
            f32x2 x1 = {o[a][i4 * 4 + 2] * inv, o[a][i4 * 4 + 3] * inv};
            bf16x2 y0 = __builtin_convertvector(x0, bf16x2);
            bf16x2 y1 = __builtin_convertvector(x1, bf16x2);
            u32x2 wv = {__builtin_bit_cast(uint32_t, y0), __builtin_bit_cast(uint32_t, y1)};
            const int chunk = a * 4 + i4;   // d = 8 chunk + 4 half .. + 3
            *(u32x2*)(row + (((chunk ^ rr) << 3) + 4 * half)) = wv;
          }
      }
      // same wave wrote and reads: the LDS operations of one wave complete in order
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int rr = (lane >> 4) + 4 * i;   // row within the pass
        const int pos = pos0 + 16 * pass + rr;
        const u32x4 v = *(const u32x4*)(stage + rr * kD + ((c16 ^ rr) << 3));
        if (pos < row1) *(u32x4*)((__bf16*)p.out + ((size_t)(qbase + pos) * p.Hq + head) * kD + c16 * 8) = v;
      }
    }
  }
}

// ---- merge of the parts of split items -----------------------------------------------------------
// One workgroup per (split item, kv head and head group, wavefront of the attention kernel); its wavefront a combines
// d = 32 a .. 32 a + 31 of that wavefront's 32 rows, each lane what the same lane of every part wrote: coalesced 1 KB reads.
// Bound by those reads (16.9 KB per part).
__global__ __launch_bounds__(256) void attn_merge_kernel(AttnParams p) {
  const int n_hg = p.Hq / p.Hkv / p.heads_per_wg, units = p.Hkv * n_hg;
  const int wave = blockIdx.x % kWaves, unit = blockIdx.x / kWaves % units, si = blockIdx.x / kWaves / units;
  if (si >= p.n_items[1]) return;
  const int4 a = ((const int4*)(p.splits + kSplitInts * si))[0];
  const int parts = p.splits[kSplitInts * si + 4];
  const int row0 = a.x, row1 = a.y, qbase = a.z, slot = a.w;
  const int lane = threadIdx.x & 63, q = threadIdx.x >> 6;
  const int pos0 = row0 + (wave / p.heads_per_wg) * kRowsPerWave;
  if (pos0 >= row1) return;
  const size_t stride = (size_t)units * kSlotFloats;   // from one part to the next
  const float* src = p.partials + ((size_t)slot * units + unit) * kSlotFloats + (size_t)wave * (64 * 66);
  float m = -INFINITY;
  for (int j = 0; j < parts; ++j) m = fmaxf(m, src[j * stride + 64 * 64 + lane]);
  float l = 0.f;
  f32x4 acc[4] = {};
#pragma unroll 4
  for (int j = 0; j < parts; ++j) {
    const float* s = src + j * stride;
    const float f = __builtin_amdgcn_exp2f(s[64 * 64 + lane] - m);
    l += f * s[64 * 65 + lane];
#pragma unroll
    for (int i4 = 0; i4 < 4; ++i4) acc[i4] += f * ((const f32x4*)s)[(q * 4 + i4) * 64 + lane];
  }
  const int row = pos0 + (lane & 31);
  if (row >= row1) return;
  const float inv = 1.0f / l;
  const int head = (unit / n_hg) * (p.Hq / p.Hkv) + (unit % n_hg) * p.heads_per_wg + wave % p.heads_per_wg;
  __bf16* dst = (__bf16*)p.out + ((size_t)(qbase + row) * p.Hq + head) * kD + 32 * q + 4 * (lane >> 5);
#pragma unroll
  for (int i4 = 0; i4 < 4; ++i4) {
    const bf16x2 y0 = __builtin_convertvector((f32x2{acc[i4][0] * inv, acc[i4][1] * inv}), bf16x2);
    const bf16x2 y1 = __builtin_convertvector((f32x2{acc[i4][2] * inv, acc[i4][3] * inv}), bf16x2);
    *(u32x2*)(dst + 8 * i4) = u32x2{__builtin_bit_cast(uint32_t, y0), __builtin_bit_cast(uint32_t, y1)};
  }
}

int heads_per_wg_for(int G) { return G % 4 == 0 ? 4 : (G % 2 == 0 ? 2 : 1); }  // divides kWaves

int check_attn(const skv_attn_desc* d) {
  if (!d) return SKV_EINVAL;
  if (d->n_q_heads < 1 || d->n_kv_heads < 1 || d->n_q_heads % d->n_kv_heads) return SKV_EINVAL;
  if (d->dtype == SKV_BF16) return d->head_dim == kD ? SKV_OK : SKV_EINVAL;
  if (d->dtype == SKV_F32) return (d->head_dim == 64 || d->head_dim == 128) ? SKV_OK : SKV_EINVAL;
  return SKV_EINVAL;
}

int64_t max_items_for(const skv_attn_desc* d, int32_t n_req, int64_t total_q_rows) {
  if (d->dtype != SKV_BF16) return 0;
  const int hpw = heads_per_wg_for(d->n_q_heads / d->n_kv_heads);
  const int pos_per_wg = (kWaves / hpw) * kRowsPerWave;
  return total_q_rows / pos_per_wg + 2 * (int64_t)n_req;   // per request: a short first tile and a ragged last one
}

// Workgroups per item, and whether a batch of this bound is small enough that its items may be split along the keys
// (with more workgroups than two rounds of the chip there is nothing to fill).
int units_of(const skv_attn_desc* d) {
  return d->n_kv_heads * (d->n_q_heads / d->n_kv_heads / heads_per_wg_for(d->n_q_heads / d->n_kv_heads));
}
int64_t max_parts_for(const skv_attn_desc* d, int64_t total_q_rows) {
  if (d->dtype != SKV_BF16) return 0;
  const int pos_per_wg = (kWaves / heads_per_wg_for(d->n_q_heads / d->n_kv_heads)) * kRowsPerWave;
  const int units = units_of(d);
  return total_q_rows / pos_per_wg * units <= kMaxSlots && units <= kCus ? kMaxSlots / units : 0;
}
size_t split_bytes(const skv_attn_desc* d, int64_t total_q_rows) {
  const int64_t parts = max_parts_for(d, total_q_rows);
  return parts ? kCus * kSplitInts * sizeof(int32_t) + (size_t)parts * units_of(d) * kSlotFloats * sizeof(float) : 0;
}

size_t zero_page_bytes(const skv_attn_desc* d) {
  return d->dtype == SKV_BF16 ? skv_align256((size_t)SKV_BLOCK_TOKENS * d->n_kv_heads * kD * 2) : 0;
}

}  // namespace

// Workspace without the area for split items: what a call needs at the least.
static size_t base_workspace(const skv_attn_desc* desc, int32_t n_req, int64_t total_q_rows) {
  const int64_t records = max_items_for(desc, n_req, total_q_rows) + max_parts_for(desc, total_q_rows);
  return 256 + zero_page_bytes(desc) + skv_align256((size_t)records * kItemInts * sizeof(int32_t));
}

extern "C" int skv_prefill_attn_workspace_size(const skv_attn_desc* desc, int32_t n_req,
                                               int64_t total_q_rows, size_t* bytes) {
  int rc = check_attn(desc);
  if (rc) return rc;
  if (n_req < 0 || total_q_rows < 0 || !bytes) return SKV_EINVAL;
  *bytes = base_workspace(desc, n_req, total_q_rows) + split_bytes(desc, total_q_rows);
  return SKV_OK;
}

// Host-checkable argument errors common to both entry points.
static int check_attn_buffers(const void* d_q, const void* d_knew, const void* d_vnew, const int32_t* d_q_off,
                              const void* d_kpool, const void* d_vpool, const int32_t* d_matched_len,
                              const int32_t* d_page_table, int32_t max_blocks, const void* d_out) {
  if (!d_q || !d_knew || !d_vnew || !d_q_off || !d_matched_len || !d_out) return SKV_EINVAL;
  if (max_blocks > 0 && (!d_page_table || !d_kpool || !d_vpool)) return SKV_EINVAL;
  if (((uintptr_t)d_q | (uintptr_t)d_knew | (uintptr_t)d_vnew | (uintptr_t)d_kpool | (uintptr_t)d_vpool |
       (uintptr_t)d_out) & 15)
    return SKV_EINVAL;
  return SKV_OK;
}

// Shared by both entry points: enqueues the schedule kernel and the attention kernel on checked arguments.
static int prefill_attn_enqueue(const skv_attn_desc* desc, int32_t n_req, const void* d_q,
                                const void* d_knew, const void* d_vnew, const int32_t* d_q_off,
                                int64_t total_q_rows, const void* d_kpool, const void* d_vpool,
                                int32_t n_pages, const int32_t* d_matched_len,
                                const int32_t* d_page_table, int32_t max_blocks, void* d_out,
                                void* d_workspace, bool may_split, void* stream) {
  hipStream_t st = (hipStream_t)stream;

  AttnParams p;
  p.q = d_q; p.knew = d_knew; p.vnew = d_vnew; p.kpool = d_kpool; p.vpool = d_vpool; p.out = d_out;
  p.q_off = d_q_off; p.matched_len = d_matched_len; p.page_table = d_page_table;
  p.n_items = (const int32_t*)d_workspace;
  p.zero_page = (const char*)d_workspace + 256;
  p.items = (const int32_t*)((char*)d_workspace + 256 + zero_page_bytes(desc));
  p.n_req = n_req; p.max_blocks = max_blocks; p.n_pages = n_pages;
  p.Hq = desc->n_q_heads; p.Hkv = desc->n_kv_heads;
  p.heads_per_wg = heads_per_wg_for(desc->n_q_heads / desc->n_kv_heads);
  p.scale = skv_softmax_scale(desc);

  if (desc->dtype == SKV_F32) {
    const SkvAttnF32Params f = {d_q, d_knew, d_vnew, d_kpool, d_vpool, d_out, d_q_off, d_matched_len, d_page_table,
                                n_req, max_blocks, n_pages, desc->n_q_heads, desc->n_kv_heads, skv_softmax_scale(desc),
                                total_q_rows};
    return skv_attn_f32_enqueue(f, desc->head_dim, stream);
  }

  const int64_t max_parts = may_split ? max_parts_for(desc, total_q_rows) : 0;
  const int64_t max_items = max_items_for(desc, n_req, total_q_rows) + max_parts;
  const int pos_per_wg = (kWaves / p.heads_per_wg) * kRowsPerWave;
  const int units = units_of(desc);
  const int64_t grid = max_items * units;
  if (grid > 0x7fffffff || max_items > 0x3fffffff) return SKV_ERANGE;
  char* const split_area = (char*)d_workspace + base_workspace(desc, n_req, total_q_rows);
  p.splits = max_parts ? (const int32_t*)split_area : nullptr;
  p.partials = max_parts ? (float*)(split_area + kCus * kSplitInts * sizeof(int32_t)) : nullptr;
  attn_schedule_kernel<<<1, kSchedThreads, 0, st>>>(n_req, d_q_off, d_matched_len, pos_per_wg, (int)max_items, units,
                                                    (int32_t*)d_workspace, (int32_t*)p.items, (int32_t*)p.splits,
                                                    (uint4*)p.zero_page, (int)(zero_page_bytes(desc) / 16));
  SKV_HIP(hipGetLastError());
  attn_bf16_kernel<<<(int)grid, kThreads, 0, st>>>(p);
  SKV_HIP(hipGetLastError());
  if (max_parts) {   // a split item has two parts at least
    attn_merge_kernel<<<(int)(max_parts / 2 * units * kWaves), 256, 0, st>>>(p);
    SKV_HIP(hipGetLastError());
  }
  return SKV_OK;
}

extern "C" int skv_prefill_attn(const skv_attn_desc* desc, int32_t n_req, const void* d_q,
                                const void* d_knew, const void* d_vnew, const int32_t* d_q_off,
                                int64_t total_q_rows, const void* d_kpool, const void* d_vpool,
                                int32_t n_pages, const int32_t* d_matched_len,
                                const int32_t* d_page_table, int32_t max_blocks, void* d_out,
                                void* d_workspace, size_t workspace_bytes, void* stream) {
  int rc = check_attn(desc);
  if (rc) return rc;
  if (n_req < 0 || total_q_rows < 0 || n_pages < 0 || max_blocks < 0) return SKV_EINVAL;
  if (n_req == 0 || total_q_rows == 0) return SKV_OK;
  rc = check_attn_buffers(d_q, d_knew, d_vnew, d_q_off, d_kpool, d_vpool, d_matched_len, d_page_table, max_blocks,
                          d_out);
  if (rc) return rc;
  size_t need = 0;
  skv_prefill_attn_workspace_size(desc, n_req, total_q_rows, &need);
  if (!d_workspace || workspace_bytes < need) return SKV_ENOMEM;
  if ((uintptr_t)d_workspace & 15) return SKV_EINVAL;
  return prefill_attn_enqueue(desc, n_req, d_q, d_knew, d_vnew, d_q_off, total_q_rows, d_kpool, d_vpool, n_pages,
                              d_matched_len, d_page_table, max_blocks, d_out, d_workspace, true, stream);
}

// ---- the same call for callers that cannot allocate ---------------------------------------------
// The work list and the page of zeros live in a file-scope device array instead of a caller workspace.  Every GPU
// the library runs on holds its own copy of the array at its own address, looked up once per device.
static __device__ __align__(256) unsigned char scratch[SKV_STATIC_SCRATCH_BYTES];

namespace {
constexpr int kMaxDevices = 64;
std::atomic<void*> g_scratch_ptr[kMaxDevices];   // device address of `scratch` per device, null until looked up

int scratch_of_current_device(void** out) {
  int dev = -1;
  SKV_HIP(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices) return SKV_ERANGE;
  void* ptr = g_scratch_ptr[dev].load(std::memory_order_acquire);
  if (!ptr) {
    // the array's name is only a host-side stand-in; this is its address on the current device
    SKV_HIP(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
    if (!ptr) return SKV_EHIP;
    g_scratch_ptr[dev].store(ptr, std::memory_order_release);   // racing first calls store the same value
  }
  *out = ptr;
  return SKV_OK;
}
}  // namespace

extern "C" int skv_prefill_attn_static(const skv_attn_desc* desc, int32_t n_req, const void* d_q,
                                       const void* d_knew, const void* d_vnew, const int32_t* d_q_off,
                                       int64_t total_q_rows, const void* d_kpool, const void* d_vpool,
                                       int32_t n_pages, const int32_t* d_matched_len,
                                       const int32_t* d_page_table, int32_t max_blocks, void* d_out,
                                       void* stream) {
  int rc = check_attn(desc);
  if (rc) return rc;
  if (n_req < 0 || total_q_rows < 0 || n_pages < 0 || max_blocks < 0) return SKV_EINVAL;
  if (n_req == 0 || total_q_rows == 0) return SKV_OK;
  rc = check_attn_buffers(d_q, d_knew, d_vnew, d_q_off, d_kpool, d_vpool, d_matched_len, d_page_table, max_blocks,
                          d_out);
  if (rc) return rc;
  if (base_workspace(desc, n_req, total_q_rows) > (size_t)SKV_STATIC_SCRATCH_BYTES)
    return SKV_ERANGE;   // batch too large for the built-in scratch
  void* ws = nullptr;
  rc = scratch_of_current_device(&ws);
  if (rc) return rc;
  // the schedule kernel rewrites the item count, the page of zeros and every record it hands out on each call,
  // so nothing of the previous call's contents is read
  return prefill_attn_enqueue(desc, n_req, d_q, d_knew, d_vnew, d_q_off, total_q_rows, d_kpool, d_vpool, n_pages,
                              d_matched_len, d_page_table, max_blocks, d_out, ws, false, stream);
}

// ---- measurement aid: what the matrix cores sustain on given operand values ----
// The clock the chip holds under matrix load depends on the values flowing through the multipliers, so the rate a
// kernel can reach is a property of its data as well as of its code.  Every wavefront keeps six (A, B) operand
// pairs of the caller's data in registers and issues the attention kernel's MFMA back to back into four
// accumulators: no memory traffic, no other instructions.  One workgroup of eight wavefronts per compute unit; its
// LDS claim keeps a second workgroup off the unit, so every SIMD runs exactly two wavefronts from start to end.
// With side work, every MFMA is accompanied by what the attention kernel's softmax issues per MFMA at the least --
// its A operand read from LDS (16 bytes per lane), one multiply-add, one exponential, one add and half a packed
// conversion -- on values that depend on nothing the matrix core produces: no dependency on a result, no global
// load, no barrier.  What this form sustains bounds any schedule of that instruction mix.
namespace {
constexpr int kRateMaxBlocks = 512, kRateThreads = 512, kRatePairs = 6, kRateLdsBytes = 96 * 1024;
template <bool kSide>
__global__ __launch_bounds__(kRateThreads) void mfma_rate_kernel(const u32x4* __restrict__ ops, float* __restrict__ sink,
                                                                 int iters) {
  __shared__ u32x4 claim[kRateLdsBytes / 16];
  const size_t lane_id = (size_t)blockIdx.x * kRateThreads + threadIdx.x;
  bf16x8 a[kRatePairs], b[kRatePairs];
#pragma unroll
  for (int i = 0; i < kRatePairs; ++i) {
    const u32x4 x = ops[(lane_id * kRatePairs + i) * 2], y = ops[(lane_id * kRatePairs + i) * 2 + 1];
    a[i] = __builtin_bit_cast(bf16x8, x);
    b[i] = __builtin_bit_cast(bf16x8, y);
  }
  f32x16 c[4];
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int e = 0; e < 16; ++e) c[j][e] = 0.f;
  float t = 0.f;
  if (kSide) {
    // the workgroup's own 96 KB of operand data fill the LDS; a wavefront reads A operands from its own 8 KB of it
    constexpr int kVecs = kRateLdsBytes / 16;
    for (int i = threadIdx.x; i < kVecs; i += kRateThreads) claim[i] = ops[(size_t)blockIdx.x * kVecs + i];
    __syncthreads();
    const uint32_t abase = lds_addr(&claim[(threadIdx.x & 63) + (threadIdx.x >> 6) * 512]);
    bf16x8 ar[4] = {a[0], a[1], a[2], a[3]};   // ring: the read behind MFMA j serves MFMA j + 4
    float x[4], e_prev = 0.f, e_pp = 0.f;
#pragma unroll
    for (int j = 0; j < 4; ++j) x[j] = (float)((threadIdx.x * 37 + j * 101) % 1000) * 0.001f;
    for (int it = 0; it < iters; ++it) {
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        lds_wait(3, ar[j & 3]);
        c[j & 3] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ar[j & 3], b[(j / 4 + j) % kRatePairs], c[j & 3], 0, 0, 0);
        ar[j & 3] = lds_read_b128(abase, (j & 7) * 1024);
        x[j & 3] = __builtin_fmaf(-1.9371f, __builtin_fabsf(x[j & 3]), 1.0f);   // bounded, never settles
        const float e = __builtin_amdgcn_exp2f(x[j & 3]);
        t += e_prev;                       // results are consumed one step late, as in the attention kernel: nothing
        if (j & 1) {                       // waits for the transcendental unit
          f32x2 pr = {e_pp, e_prev};
          const bf16x2 cv = __builtin_convertvector(pr, bf16x2);
          asm volatile("" ::"v"(cv));
        }
        e_pp = e_prev;
        e_prev = e;
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    lds_wait(0, ar[0], ar[1], ar[2], ar[3]);
  } else {
    for (int it = 0; it < iters; ++it) {
#pragma unroll
      for (int j = 0; j < 16; ++j)
        c[j & 3] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[j % kRatePairs], b[(j / 4 + j) % kRatePairs], c[j & 3], 0, 0, 0);
    }
  }
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int e = 0; e < 16; ++e) t += c[j][e];
  volatile uint32_t* used = (volatile uint32_t*)claim;   // the array has to be used to be allocated
  used[threadIdx.x] = __float_as_uint(t);
  sink[lane_id] = __uint_as_float(used[threadIdx.x]);
}
}  // namespace

extern "C" int skv_mfma_rate(const void* d_operands, size_t operand_bytes, int32_t iters, int32_t side_work,
                             float* d_sink, size_t sink_bytes, double* flops, void* stream) {
  if (!d_operands || !d_sink || iters < 1 || ((uintptr_t)d_operands & 15)) return SKV_EINVAL;
  if (side_work != 0 && side_work != 1) return SKV_EINVAL;
  if (operand_bytes < SKV_MFMA_RATE_OPERAND_BYTES || sink_bytes < SKV_MFMA_RATE_SINK_BYTES) return SKV_ENOMEM;
  int dev = 0, cus = 0;
  SKV_HIP(hipGetDevice(&dev));
  SKV_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
  const int blocks = cus < kRateMaxBlocks ? cus : kRateMaxBlocks;
  if (side_work)
    mfma_rate_kernel<true><<<blocks, kRateThreads, 0, (hipStream_t)stream>>>((const u32x4*)d_operands, d_sink, iters);
  else
    mfma_rate_kernel<false><<<blocks, kRateThreads, 0, (hipStream_t)stream>>>((const u32x4*)d_operands, d_sink, iters);
  SKV_HIP(hipGetLastError());
  if (flops) *flops = (double)blocks * (kRateThreads / 64) * (double)iters * 16.0 * (2.0 * 32 * 32 * 16);
  return SKV_OK;
}
