// The page copy of the gather, for the kernels that carry it: alone, or beside other work of the same step.
#ifndef SKV_GATHER_H
#define SKV_GATHER_H
#include "skv_internal.h"

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

struct SkvGather {
  int n_req;
  const u32x4 *kpool, *vpool;
  int n_pages;
  const int32_t *matched_len, *page_table;
  int max_blocks;
  int64_t* ctx_off;
  u32x4 *kctx, *vctx;
  int64_t cap_pages;
  int page_vec;   // 16-byte vectors per page
  int slices_log; // logarithm of the workgroups per page
  bool large;     // a copy with a launch of its own
};
constexpr int kSkvGatherScan = 512;   // requests up to which every workgroup scans the matched lengths itself

// Counter updates that a lookup left for a later kernel (skv_match_window): those of the matched blocks' records.
struct SkvCount {
  uint32_t* ctr;
  size_t ctr_plane;
  const int32_t *records, *req_tenant, *matched_len;   // records null: nothing is left
  int max_blocks, n_req;
};

// Arguments checked and laid out; workgroups of a call; the call.  d_q_off: the suffix offsets are written too; count: and those counters.
int skv_gather_check(const skv_attn_desc* desc, int32_t n_req, const void* d_kpool, const void* d_vpool, int32_t n_pages,
                     const int32_t* d_matched_len, const int32_t* d_page_table, int32_t max_blocks, int64_t* d_ctx_off, void* d_kctx,
                     void* d_vctx, int64_t ctx_capacity_tokens, SkvGather* g);
int skv_gather_blocks(const SkvGather& g);
int skv_gather_enqueue(const SkvGather& g, bool beside, const int32_t* d_req_off, int32_t* d_q_off, const SkvCount& count, void* stream);
int skv_count_enqueue(const SkvCount& count, void* stream);

// ---- fp32 prefill attention (skv_attn_f32.hip), enqueued by skv_prefill_attn and skv_prefill_step on checked arguments ----
struct SkvAttnF32Params {
  const void *q, *knew, *vnew, *kpool, *vpool;
  void* out;
  const int32_t *q_off, *matched_len, *page_table;
  int n_req, max_blocks, n_pages, Hq, Hkv;
  float scale;
  int64_t max_rows;          // rows of q and out
  const int32_t* req_off;    // of a launch that writes q_off (the enqueuing function's choice): what that is made from
};
// The rest of a step, with the attention or in front of it: suffix offsets, pages, counters.
struct SkvStepRest {
  const SkvGather* gather;
  const int32_t* req_off;
  int32_t* q_off;
  const SkvCount* count;
};
int skv_attn_f32_enqueue(const SkvAttnF32Params& p, int head_dim, const SkvStepRest* rest, void* stream);

#ifdef __HIPCC__
// Request r's: a workgroup.
__device__ __forceinline__ void skv_count_request(const SkvCount& c, int r) {
  const int n = min(max(c.matched_len[r], 0) / SKV_BLOCK_TOKENS, c.max_blocks), tenant = c.req_tenant[r];
  if (n <= 0) return;   // (only a tenant of the tree has matched anything)
  uint32_t* const tenants = c.ctr + (size_t)(1 + (tenant >> 5)) * c.ctr_plane;
  for (int i = threadIdx.x; i < n; i += blockDim.x) {
    const int blk = c.records[(size_t)r * c.max_blocks + i];
    atomicAdd(c.ctr + blk, 1u);
    atomicOr(tenants + blk, 1u << (tenant & 31));
  }
}

// What workgroup `block` of n_blocks copies (n_blocks is a multiple of the slices; kSliced: a page may have several): it loops over the
// global list of matched pages, each moving as 16-byte vectors with all loads of a step issued before its stores.  kScan: the workgroup scans the matched lengths
// itself (the first one also writes the offsets) and finds the owner of a page in `first`, kSkvGatherScan + 1 places in LDS.
// (The pointers as arguments: only there does __restrict__ tell the compiler that the copies leave offsets and table alone, so that it
// reads these with scalar loads.  Of 599 requests, 23490 pages of 4 KB: 75 us, 115 with vector loads.  Slices known at run time only
// cost calls without any up to a tenth: 860 pages of 32 KB 19.0 us, 21.9 with two divisions for them, 21.0 with shifts.)
template <bool kScan, bool kSliced, int kThreads, int kUnroll>
__device__ __forceinline__ void skv_gather_pages(const SkvGather& g, int block, int n_blocks, int64_t* first, const u32x4* __restrict__ kpool,
                                                 const u32x4* __restrict__ vpool, const int32_t* __restrict__ matched_len,
                                                 const int32_t* __restrict__ page_table, int64_t* __restrict__ ctx_off,
                                                 u32x4* __restrict__ kctx, u32x4* __restrict__ vctx) {
  const int n_req = g.n_req;
  int64_t total;
  if constexpr (kScan) {
    __shared__ int64_t red[kThreads / 64];
    const int own = (n_req + kThreads - 1) / kThreads;         // requests per thread
    const int r0 = min((int)threadIdx.x * own, n_req), r1 = min(r0 + own, n_req);
    auto pages_of = [&](int r) { return max(matched_len[r], 0) / SKV_BLOCK_TOKENS; };
    int64_t mine = 0;
    for (int r = r0; r < r1; ++r) mine += pages_of(r);
    int64_t at = skv_block_scan<kThreads>(mine, red, total) - mine;
    for (int r = r0; r < r1; ++r) {
      first[r] = at;
      at += pages_of(r);
      if (block == 0) ctx_off[r + 1] = at * SKV_BLOCK_TOKENS;
    }
    if (threadIdx.x == 0) {
      first[n_req] = total;
      if (block == 0) ctx_off[0] = 0;
    }
    __syncthreads();
  } else {
    total = ctx_off[n_req] / SKV_BLOCK_TOKENS;
  }
  auto pages_before = [&](int r) { return kScan ? first[r] : ctx_off[r] / SKV_BLOCK_TOKENS; };
  const int64_t end = min(total, g.cap_pages);
  const int log = kSliced ? g.slices_log : 0, slice = block & ((1 << log) - 1), per_slice = g.page_vec >> log;
  const int v0 = per_slice * slice, v1 = (slice + 1) >> log ? g.page_vec : v0 + per_slice;   // (the last takes the rest)
  for (int64_t p = block >> log; p < end; p += n_blocks >> log) {
    // request that owns output page p: the last one with no more than p pages before it
    int lo = 0, hi = n_req;  // invariant: pages_before(lo) <= p < pages_before(hi)
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (pages_before(mid) <= p) lo = mid; else hi = mid;
    }
    const int64_t before = pages_before(lo);
    const int j = (int)(p - before);
    if (j >= g.max_blocks) continue;
    const int page = page_table[(size_t)lo * g.max_blocks + j];
    if (page < 0 || page >= g.n_pages) continue;  // uniform per workgroup
    const u32x4* ks = kpool + (size_t)page * g.page_vec;
    const u32x4* vs = vpool + (size_t)page * g.page_vec;
    u32x4* kd = kctx + (size_t)p * g.page_vec;
    u32x4* vd = vctx + (size_t)p * g.page_vec;
    for (int base = v0; base < v1; base += kThreads * kUnroll) {
      u32x4 a[kUnroll], b[kUnroll];
#pragma unroll
      for (int u = 0; u < kUnroll; ++u) {
        const int i = base + u * kThreads + threadIdx.x;
        if (i < v1) {
          a[u] = __builtin_nontemporal_load(ks + i);
          b[u] = __builtin_nontemporal_load(vs + i);
        }
      }
#pragma unroll
      for (int u = 0; u < kUnroll; ++u) {
        const int i = base + u * kThreads + threadIdx.x;
        if (i < v1) {
          __builtin_nontemporal_store(a[u], kd + i);
          __builtin_nontemporal_store(b[u], vd + i);
        }
      }
    }
  }
}

// The same copy without LDS of its own and in few registers: beside a kernel that holds most of both, or in its launch.  (There every workgroup has the
// kernel's LDS, 80 to 128 KB of the bf16 attention's: it waits until a compute unit, or half of one, is free.)  Up to kSkvGatherScan
// requests; workgroup `block` of n_blocks takes whole pages; the first one writes the offsets.
template <int kThreads, int kUnroll>
__device__ __forceinline__ void skv_copy_pages(int n_req, const char* __restrict__ kpool, const char* __restrict__ vpool, int n_pages,
                                               const int32_t* __restrict__ matched_len, const int32_t* __restrict__ page_table, int max_blocks,
                                               int64_t* __restrict__ ctx_off, char* __restrict__ kctx, char* __restrict__ vctx,
                                               int64_t cap_pages, int page_bytes, int block, int n_blocks) {
  // A lane holds the pages before its `per` requests.  Nothing in LDS: two attention workgroups of four wavefronts leave none of it.
  const int lane = threadIdx.x & 63, per = (n_req + 63) / 64;
  auto pages_of = [&](int r) __attribute__((always_inline)) { return max(matched_len[r], 0) / SKV_BLOCK_TOKENS; };
  const int r0 = min(lane * per, n_req), r1 = min(r0 + per, n_req);
  int64_t before = 0, end;
  {
    for (int r = r0; r < r1; ++r) before += pages_of(r);
    const int64_t own = before;
    before = skv_wave_scan(before);
    end = min(skv_lane(before, 63), cap_pages);
    before -= own;
    if (block == 0 && threadIdx.x < 64) {
      int64_t at = before;
      if (lane == 0) ctx_off[0] = 0;
      for (int r = r0; r < r1; ++r) {
        at += pages_of(r);
        ctx_off[r + 1] = at * SKV_BLOCK_TOKENS;
      }
    }
  }
  const unsigned at = threadIdx.x * 16;
  // Page ids are asked for a page ahead: one workgroup per compute unit has nobody to cover the read.
  int r = 0, n = 0;      // request that owns the page, its pages
  int64_t first = 0;     // and the pages before it
  auto page_of = [&](int64_t p) __attribute__((always_inline)) {
    if (p >= end) return -1;
    if (p >= first + n) {   // (it does end: p < end)
      const int l = __builtin_popcountll(__ballot(before <= p)) - 1;   // the last lane with no more than p pages before it
      r = l * per;
      first = skv_lane(before, l);
      for (n = pages_of(r); p >= first + n; n = pages_of(r)) {
        first += n;
        ++r;
      }
    }
    const int64_t j = p - first;
    return j < max_blocks ? page_table[(size_t)r * max_blocks + j] : -1;
  };
  int next = page_of(block);
  for (int64_t p = block; p < end; p += n_blocks) {
    const int page = __builtin_amdgcn_readfirstlane(next);
    next = page_of(p + n_blocks);
    if (page < 0 || page >= n_pages) continue;
    const __amdgpu_buffer_rsrc_t ks = __builtin_amdgcn_make_buffer_rsrc((void*)(kpool + (size_t)page * page_bytes), 0, page_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t vs = __builtin_amdgcn_make_buffer_rsrc((void*)(vpool + (size_t)page * page_bytes), 0, page_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t kd = __builtin_amdgcn_make_buffer_rsrc((void*)(kctx + (size_t)p * page_bytes), 0, page_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t vd = __builtin_amdgcn_make_buffer_rsrc((void*)(vctx + (size_t)p * page_bytes), 0, page_bytes, 0x00020000);
    constexpr int kStep = kThreads * 16;
    for (int base = 0; base < page_bytes; base += kUnroll * kStep) {
      u32x4 a[kUnroll], b[kUnroll];
#pragma unroll
      for (int u = 0; u < kUnroll; ++u) {   // (2: non-temporal; a step begins inside the page, so the range check holds)
        if (base + u * kStep >= page_bytes) break;
        a[u] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(ks, at, base + u * kStep, 2));
        b[u] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(vs, at, base + u * kStep, 2));
      }
#pragma unroll
      for (int u = 0; u < kUnroll; ++u) {
        if (base + u * kStep >= page_bytes) break;
        __builtin_amdgcn_raw_buffer_store_b128(a[u], kd, at, base + u * kStep, 2);
        __builtin_amdgcn_raw_buffer_store_b128(b[u], vd, at, base + u * kStep, 2);
      }
    }
  }
}
#endif
#endif
