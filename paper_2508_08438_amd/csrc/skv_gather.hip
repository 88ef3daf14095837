// Page-table gather of the reused KV pages into per-request contiguous staging.
//
// SafeKV Section 4.3.2: after the lookup stops at a compressed node the required KV blocks are
// read directly from its address vector.  Here the address vector is the page table written by
// the match; a page is one contiguous chunk of 16 * n_kv_heads * head_dim elements, so the
// gather is a batch of page-sized copies chosen by the table (the copy itself: skv_gather_pages).
#include <algorithm>

#include "skv_gather.h"

namespace {

constexpr int kThreads = 256;
constexpr int kUnroll = 8;  // 16-byte vectors in flight per thread and pool

// Where the output of every request starts, one workgroup.
constexpr int kOffThreads = 1024, kOffPer = 4;
__global__ __launch_bounds__(kOffThreads) void ctx_offsets_kernel(int n_req, const int32_t* __restrict__ matched_len,
                                                                  int64_t* __restrict__ ctx_off) {
  __shared__ int64_t red[kOffThreads / 64];
  int64_t carry = 0;
  if (threadIdx.x == 0) ctx_off[0] = 0;
  for (int64_t base = 0; base < n_req; base += kOffThreads * kOffPer) {
    const int64_t r0 = base + threadIdx.x * kOffPer;
    int64_t v[kOffPer], own = 0, total;
#pragma unroll
    for (int k = 0; k < kOffPer; ++k) v[k] = r0 + k < n_req ? max(matched_len[r0 + k], 0) / SKV_BLOCK_TOKENS : 0;
#pragma unroll
    for (int k = 0; k < kOffPer; ++k) own += v[k];
    int64_t x = carry + skv_block_scan<kOffThreads>(own, red, total) - own;
    carry += total;
#pragma unroll
    for (int k = 0; k < kOffPer; ++k) {
      x += v[k];
      if (r0 + k < n_req) ctx_off[r0 + k + 1] = x * SKV_BLOCK_TOKENS;
    }
  }
}

// A kernel for the offsets in front of it (kScan false) costs a launch, 4.5 us for one request, but reads the lengths once: one page
// each of 16 / 256 / 512 requests 14.0 / 19.4 / 23.5 us scanned, 16.6 / 22.0 / 24.4 with that kernel; of 1024 / 4096 / 16384 33.6 /
// 158 / 685 scanned, 33.7 / 113 / 432 with it; 40 pages each of 1024 1053 and 1044.
// kOffsets: the first workgroup writes the suffix offsets instead (skv_suffix_offsets of up to kSkvGatherScan requests), which
// neither reads nor delays a page: one launch less in a step.  n_count workgroups behind it update the counters of a request each.
template <bool kScan, bool kOffsets, bool kSliced>
__global__ __launch_bounds__(kThreads) void gather_pages_kernel(SkvGather g, const int32_t* __restrict__ req_off, int32_t* __restrict__ q_off,
                                                                SkvCount count, int n_count) {
  if constexpr (kOffsets) {
    if (blockIdx.x == 0) {
      __shared__ int red[kThreads / 64];
      constexpr int kPer = kSkvGatherScan / kThreads;
      int v[kPer], own = 0, total;
      const int r0 = threadIdx.x * kPer;
#pragma unroll
      for (int k = 0; k < kPer; ++k) own += v[k] = r0 + k < g.n_req ? max(0, req_off[r0 + k + 1] - req_off[r0 + k] - g.matched_len[r0 + k]) : 0;
      int x = skv_block_scan<kThreads>(own, red, total) - own;
      if (threadIdx.x == 0) q_off[0] = 0;
#pragma unroll
      for (int k = 0; k < kPer; ++k) {
        x += v[k];
        if (r0 + k < g.n_req) q_off[r0 + k + 1] = x;
      }
      return;
    }
    if ((int)blockIdx.x <= n_count) return skv_count_request(count, (int)blockIdx.x - 1);
  }
  __shared__ int64_t first[kScan ? kSkvGatherScan + 1 : 1];
  const int others = kOffsets ? 1 + n_count : 0;
  skv_gather_pages<kScan, kSliced, kThreads, kUnroll>(g, (int)blockIdx.x - others, (int)gridDim.x - others, first, g.kpool, g.vpool,
                                                      g.matched_len, g.page_table, g.ctx_off, g.kctx, g.vctx);
}

__global__ __launch_bounds__(kThreads) void count_matched_kernel(SkvCount count) { skv_count_request(count, blockIdx.x); }

// The same copy for a call that runs beside a kernel which holds most of the chip's registers (prefill attention: 240 of a
// SIMD's 512 for each of two wavefronts): one workgroup per compute unit with one wavefront per SIMD in the 32 registers that
// are left, and none of the LDS, which two of its workgroups may fill (with 4 KB for a scan of the offsets instead of the lanes it had
// to wait for one of them to end, and they for it: 335 MB beside 50 us of attention 268 us, now 110), so it needs no compute unit of its
// own and takes what the other kernel leaves of the memory's time.  Addresses are
// buffer descriptors and scalar offsets for the registers' sake; what lies behind a page's end is neither read nor written.
// Alone it is the faster form of a large copy too: one workgroup per compute unit keeps enough in flight and goes through neighbouring
// pages together.  us of the plain form / of this one, 32 KB pages 1024 24.8 / 25.8, 2048 51.5 / 47.6, 4096 101 / 93, 16384 401 / 379 (5.67
// TB/s); 16 KB 2048 26.9 / 26.1, 16384 197 / 184; but 8 KB of 253 requests, 22500 pages, 74.2 / 78.3; 4 KB 16384 52.6 / 68.0.  Only for
// callers that know how full their staging is: skv_gather_kv knows its size alone, and 822 pages of 382 requests in one for 24660 take
// 19.8 / 24.2, 520 of 104 14.5 / 16.5.
constexpr int kPref = kSkvGatherScan;
constexpr int kBesideGrid = 256, kBesideUnroll = 3;
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_num_vgpr(32))) void gather_beside_kernel(
    int n_req, const char* __restrict__ kpool, const char* __restrict__ vpool, int n_pages,
    const int32_t* __restrict__ matched_len, const int32_t* __restrict__ page_table, int max_blocks,
    int64_t* __restrict__ ctx_off, char* __restrict__ kctx, char* __restrict__ vctx, int64_t cap_pages, int page_bytes) {
  skv_copy_pages<kThreads, kBesideUnroll>(n_req, kpool, vpool, n_pages, matched_len, page_table, max_blocks, ctx_off, kctx, vctx, cap_pages, page_bytes,
                                          (int)blockIdx.x, kBesideGrid);
}

// Inverse of the gather: one workgroup per (request, new block) slot of the table, persistent grid.
__global__ __launch_bounds__(kThreads) void scatter_pages_kernel(
    int n_req, const u32x4* __restrict__ knew, const u32x4* __restrict__ vnew, const int32_t* __restrict__ q_off,
    const int32_t* __restrict__ new_pages, int max_new_blocks, u32x4* __restrict__ kpool, u32x4* __restrict__ vpool,
    int n_pages, int page_vec) {
  const int64_t slots = (int64_t)n_req * max_new_blocks;
  for (int64_t sidx = blockIdx.x; sidx < slots; sidx += gridDim.x) {
    const int r = (int)(sidx / max_new_blocks), j = (int)(sidx % max_new_blocks);
    const int page = new_pages[sidx];
    const int qb = q_off[r];
    const int full = (q_off[r + 1] - qb) / SKV_BLOCK_TOKENS;
    if (page < 0 || page >= n_pages || j >= full) continue;  // uniform per workgroup
    const size_t src = ((size_t)qb + (size_t)j * SKV_BLOCK_TOKENS) * (page_vec / SKV_BLOCK_TOKENS);  // 16-byte vectors per row
    const u32x4* ks = knew + src;
    const u32x4* vs = vnew + src;
    u32x4* kd = kpool + (size_t)page * page_vec;
    u32x4* vd = vpool + (size_t)page * page_vec;
    for (int base = 0; base < page_vec; base += kThreads * kUnroll) {
      u32x4 a[kUnroll], b[kUnroll];
#pragma unroll
      for (int u = 0; u < kUnroll; ++u) {
        const int i = base + u * kThreads + threadIdx.x;
        if (i < page_vec) {
          a[u] = __builtin_nontemporal_load(ks + i);
          b[u] = __builtin_nontemporal_load(vs + i);
        }
      }
#pragma unroll
      for (int u = 0; u < kUnroll; ++u) {
        const int i = base + u * kThreads + threadIdx.x;
        if (i < page_vec) {
          __builtin_nontemporal_store(a[u], kd + i);
          __builtin_nontemporal_store(b[u], vd + i);
        }
      }
    }
  }
}

// Plain streaming copy, same vector width and loads-before-stores shape as the page copies above.
__global__ __launch_bounds__(kThreads) void stream_copy_kernel(const u32x4* __restrict__ src, u32x4* __restrict__ dst,
                                                               int64_t n_vec) {
  const int64_t stride = (int64_t)gridDim.x * kThreads * kUnroll;
  for (int64_t base = (int64_t)blockIdx.x * kThreads * kUnroll; base < n_vec; base += stride) {
    u32x4 a[kUnroll];
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
      const int64_t i = base + (int64_t)u * kThreads + threadIdx.x;
      if (i < n_vec) a[u] = __builtin_nontemporal_load(src + i);
    }
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
      const int64_t i = base + (int64_t)u * kThreads + threadIdx.x;
      if (i < n_vec) __builtin_nontemporal_store(a[u], dst + i);
    }
  }
}

// What a step does not let the merge of split items carry.
bool large_copy(int64_t pages, int64_t page_bytes) { return page_bytes >= 16384 && pages * page_bytes >= (48 << 20); }
// Workgroups per page: where a batch has no page for every compute unit a page of 32 KB is several workgroups' worth of loads in
// flight.  us with 1 / 2 / 4 slices: 16 pages 4.95 / 4.1 / 3.8, 128 (of the fp32 pool's 32 KB) 6.4 / 5.6 / 5.3, 187 6.3 / 5.9 / 6.2,
// 512 11.9 / 12.3 / 14.1.
int slices_log_for(int64_t pages) { return pages <= 128 ? 2 : pages <= 256 ? 1 : 0; }

}  // namespace

extern "C" int skv_stream_copy(void* d_dst, const void* d_src, size_t bytes, void* stream) {
  if (bytes == 0) return SKV_OK;
  if (!d_dst || !d_src || (bytes & 15) || (((uintptr_t)d_dst | (uintptr_t)d_src) & 15)) return SKV_EINVAL;
  const int64_t n_vec = (int64_t)(bytes / 16);
  const int64_t per_wg = (int64_t)kThreads * kUnroll;
  const int64_t want = (n_vec + per_wg - 1) / per_wg;
  stream_copy_kernel<<<(int)(want < 256 * 16 ? want : 256 * 16), kThreads, 0, (hipStream_t)stream>>>(
      (const u32x4*)d_src, (u32x4*)d_dst, n_vec);
  SKV_HIP(hipGetLastError());
  return SKV_OK;
}

extern "C" int skv_scatter_kv(const skv_attn_desc* desc, int32_t n_req, const void* d_knew, const void* d_vnew,
                              const int32_t* d_q_off, const int32_t* d_new_pages, int32_t max_new_blocks,
                              void* d_kpool, void* d_vpool, int32_t n_pages, void* stream) {
  if (!desc || n_req < 0 || n_pages < 0 || max_new_blocks < 0) return SKV_EINVAL;
  if (desc->dtype != SKV_F32 && desc->dtype != SKV_BF16) return SKV_EINVAL;
  if (desc->n_kv_heads < 1 || desc->head_dim < 1) return SKV_EINVAL;
  const int64_t row_bytes = (int64_t)desc->n_kv_heads * desc->head_dim * (desc->dtype == SKV_F32 ? 4 : 2);
  if (row_bytes % 16 || row_bytes * SKV_BLOCK_TOKENS / 16 > 0x7fffffff) return SKV_EINVAL;
  if (n_req == 0 || max_new_blocks == 0) return SKV_OK;
  if (!d_knew || !d_vnew || !d_q_off || !d_new_pages || !d_kpool || !d_vpool) return SKV_EINVAL;
  if (((uintptr_t)d_kpool | (uintptr_t)d_vpool | (uintptr_t)d_knew | (uintptr_t)d_vnew) & 15) return SKV_EINVAL;
  const int64_t slots = (int64_t)n_req * max_new_blocks;
  const int grid = (int)(slots < 256 * 16 ? slots : 256 * 16);
  scatter_pages_kernel<<<grid, kThreads, 0, (hipStream_t)stream>>>(
      n_req, (const u32x4*)d_knew, (const u32x4*)d_vnew, d_q_off, d_new_pages, max_new_blocks, (u32x4*)d_kpool,
      (u32x4*)d_vpool, n_pages, (int)(row_bytes * SKV_BLOCK_TOKENS / 16));
  SKV_HIP(hipGetLastError());
  return SKV_OK;
}

int skv_gather_check(const skv_attn_desc* desc, int32_t n_req, const void* d_kpool, const void* d_vpool, int32_t n_pages,
                     const int32_t* d_matched_len, const int32_t* d_page_table, int32_t max_blocks, int64_t* d_ctx_off, void* d_kctx,
                     void* d_vctx, int64_t ctx_capacity_tokens, SkvGather* g) {
  if (!desc || n_req < 0 || n_pages < 0 || max_blocks < 0 || ctx_capacity_tokens < 0) return SKV_EINVAL;
  if (desc->dtype != SKV_F32 && desc->dtype != SKV_BF16) return SKV_EINVAL;
  if (desc->n_kv_heads < 1 || desc->head_dim < 1) return SKV_EINVAL;
  const int64_t page_bytes = (int64_t)SKV_BLOCK_TOKENS * desc->n_kv_heads * desc->head_dim *
                             (desc->dtype == SKV_F32 ? 4 : 2);
  if (page_bytes % 16 || page_bytes / 16 > 0x7fffffff) return SKV_EINVAL;
  if (!d_ctx_off) return SKV_EINVAL;
  if (n_req > 0 && (!d_matched_len || !d_kpool || !d_vpool || !d_kctx || !d_vctx)) return SKV_EINVAL;
  if (n_req > 0 && max_blocks > 0 && !d_page_table) return SKV_EINVAL;
  if (((uintptr_t)d_kpool | (uintptr_t)d_vpool | (uintptr_t)d_kctx | (uintptr_t)d_vctx) & 15) return SKV_EINVAL;
  // pages the batch can move at most: what the table holds and, often far less (private blocks end a match early), what the staging does
  const int64_t upper = std::min((int64_t)n_req * max_blocks, ctx_capacity_tokens / SKV_BLOCK_TOKENS);
  *g = {n_req, (const u32x4*)d_kpool, (const u32x4*)d_vpool, n_pages, d_matched_len, d_page_table, max_blocks, d_ctx_off,
        (u32x4*)d_kctx, (u32x4*)d_vctx, n_req && max_blocks ? ctx_capacity_tokens / SKV_BLOCK_TOKENS : 0, (int)(page_bytes / 16),
        n_req <= kPref ? slices_log_for(upper) : 0, large_copy(upper, page_bytes)};
  return SKV_OK;
}

int skv_gather_blocks(const SkvGather& g) {
  const int64_t upper = std::min((int64_t)g.n_req * g.max_blocks, g.cap_pages);
  return (int)(upper < 1 ? 1 : (upper < 256 * 16 ? upper : 256 * 16)) << g.slices_log;
}

int skv_count_enqueue(const SkvCount& count, void* stream) {
  if (!count.records || count.n_req == 0) return SKV_OK;
  count_matched_kernel<<<count.n_req, kThreads, 0, (hipStream_t)stream>>>(count);
  SKV_HIP(hipGetLastError());
  return SKV_OK;
}

int skv_gather_enqueue(const SkvGather& g, bool beside, const int32_t* d_req_off, int32_t* d_q_off, const SkvCount& count, void* stream) {
  hipStream_t st = (hipStream_t)stream;
  const bool scan = g.n_req <= kPref;
  beside = beside && scan && (int64_t)g.page_vec * 16 <= 0x7fffffff;
  if (scan && !beside && d_q_off) {
    const int n_count = count.records ? g.n_req : 0;
    const auto kernel = g.slices_log ? gather_pages_kernel<true, true, true> : gather_pages_kernel<true, true, false>;
    kernel<<<1 + n_count + skv_gather_blocks(g), kThreads, 0, st>>>(g, d_req_off, d_q_off, count, n_count);
    SKV_HIP(hipGetLastError());
    return SKV_OK;
  }
  int rc = d_q_off ? skv_suffix_offsets(g.n_req, d_req_off, g.matched_len, d_q_off, stream) : SKV_OK;
  if (rc == SKV_OK) rc = skv_count_enqueue(count, stream);
  if (rc) return rc;
  if (beside) {
    gather_beside_kernel<<<kBesideGrid, kThreads, 0, st>>>(
        g.n_req, (const char*)g.kpool, (const char*)g.vpool, g.n_pages, g.matched_len, g.page_table, g.max_blocks, g.ctx_off,
        (char*)g.kctx, (char*)g.vctx, g.cap_pages, g.page_vec * 16);
  } else if (scan) {
    const auto kernel = g.slices_log ? gather_pages_kernel<true, false, true> : gather_pages_kernel<true, false, false>;
    kernel<<<skv_gather_blocks(g), kThreads, 0, st>>>(g, nullptr, nullptr, count, 0);
  } else {
    ctx_offsets_kernel<<<1, kOffThreads, 0, st>>>(g.n_req, g.matched_len, g.ctx_off);
    SKV_HIP(hipGetLastError());
    if (g.max_blocks == 0) return SKV_OK;
    gather_pages_kernel<false, false, false><<<skv_gather_blocks(g), kThreads, 0, st>>>(g, nullptr, nullptr, count, 0);
  }
  SKV_HIP(hipGetLastError());
  return SKV_OK;
}

static int gather_call(const skv_attn_desc* desc, int32_t n_req, const void* d_kpool, const void* d_vpool, int32_t n_pages,
                       const int32_t* d_matched_len, const int32_t* d_page_table, int32_t max_blocks, int64_t* d_ctx_off, void* d_kctx,
                       void* d_vctx, int64_t ctx_capacity_tokens, bool beside, void* stream) {
  SkvGather g;
  const int rc = skv_gather_check(desc, n_req, d_kpool, d_vpool, n_pages, d_matched_len, d_page_table, max_blocks, d_ctx_off, d_kctx,
                                  d_vctx, ctx_capacity_tokens, &g);
  return rc ? rc : skv_gather_enqueue(g, beside, nullptr, nullptr, SkvCount{}, stream);
}

extern "C" int skv_gather_kv(const skv_attn_desc* desc, int32_t n_req, const void* d_kpool, const void* d_vpool,
                             int32_t n_pages, const int32_t* d_matched_len, const int32_t* d_page_table, int32_t max_blocks,
                             int64_t* d_ctx_off, void* d_kctx, void* d_vctx, int64_t ctx_capacity_tokens, void* stream) {
  return gather_call(desc, n_req, d_kpool, d_vpool, n_pages, d_matched_len, d_page_table, max_blocks, d_ctx_off, d_kctx, d_vctx,
                        ctx_capacity_tokens, false, stream);
}

extern "C" int skv_gather_kv_beside(const skv_attn_desc* desc, int32_t n_req, const void* d_kpool, const void* d_vpool,
                                    int32_t n_pages, const int32_t* d_matched_len, const int32_t* d_page_table,
                                    int32_t max_blocks, int64_t* d_ctx_off, void* d_kctx, void* d_vctx,
                                    int64_t ctx_capacity_tokens, void* stream) {
  return gather_call(desc, n_req, d_kpool, d_vpool, n_pages, d_matched_len, d_page_table, max_blocks, d_ctx_off, d_kctx, d_vctx,
                        ctx_capacity_tokens, true, stream);
}
