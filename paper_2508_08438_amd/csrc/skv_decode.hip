// Decode-step attention over the paged KV cache: one query token per request attends to every cached token.
//
// SafeKV Section 2.1 (the decode phase reads the cached K/V of all earlier tokens at every step; KV reuse
// changes where those pages come from, not what is computed).  The kernel reads the same pools through the
// same page table as the prefill kernel.  A step moves every cached K and V byte once and does 4*d flops per
// byte pair, so it is HBM bound; every workgroup takes an equal share of the batch's key tiles, whatever requests
// they belong to, and a second kernel merges the partial softmax states of the requests that were cut.
//
// Layout of the products (MFMA 16x16): S^T = K Q^T with the G query heads of the kv head as the 16 columns,
// so one wavefront scores 16 keys for all heads with four v_mfma_f32_16x16x32_bf16; the accumulator registers
// (lane = head, registers = 4 keys) are, after exponentiation, the B operand of O^T += V^T P^T
// (v_mfma_f32_16x16x16_bf16), whose A operand comes from the LDS transpose load.
#include <algorithm>

#include "skv_internal.h"

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

constexpr int kD = 128;
constexpr int kBN = 64;               // keys per LDS tile: 16 per wavefront
constexpr int kWaves = 4;
constexpr int kThreads = kWaves * 64;
constexpr int kStages = 2;
constexpr int kKsStride = kD + 8;     // bf16 elements per K row in LDS (conflict-free b128 reads)
constexpr int kVsStride = kD + 32;    // bf16 elements per V row in LDS (conflict-free transpose loads)
constexpr int kMaxG = 16;             // query heads per kv head (the columns of one MFMA tile)
constexpr int kSlots = 512;           // workgroups that run at once: two per compute unit
constexpr float kLog2e = 1.4426950408889634f;

struct DecParams {
  const void *q, *kpool, *vpool;
  void* out;
  const int32_t *ctx_len, *page_table;
  int4* cuts;                       // [n_cuts] a request that was cut (-1: none), its first and end tile, all tiles
  float *part_m, *part_l, *part_o;  // [2 * n_shares][Hkv][G] (x d for part_o)
  int n_req, max_blocks, n_pages, Hq, Hkv, G;
  int n_shares;                     // workgroups per kv head the tiles are dealt to; 0: one workgroup per request
  int n_cuts;                       // n_req: by request; n_shares - 1 where that is less: by the share of the first piece
  float scale;
};

__device__ inline int tiles_of(const DecParams& p, int r) {
  return (max(0, min(p.ctx_len[r], p.max_blocks * SKV_BLOCK_TOKENS)) + kBN - 1) / kBN;
}
// T tiles dealt to n shares: the first T % n shares hold one tile more than the others.
__device__ inline int share_begin(int i, int T, int n) { return i * (T / n) + min(i, T % n); }
__device__ inline int share_of(int tile, int T, int n) {
  const int q = T / n, big = T % n * (q + 1);
  return tile < big ? tile / (q + 1) : T % n + (tile - big) / q;
}

// A share of a kv head is a run of the T tiles of the batch, request after request, about T / n of them: every
// workgroup streams the same number of bytes whatever the contexts' lengths, in one round over the chip, and pays its
// start-up once.  A request wholly inside a share is finished there; of the others every share holds one piece, and a share
// cuts two requests at most: the one it begins in (slot 2 i) and the one it ends in (slot 2 i + 1).
// Bound by HBM: 64 requests of 4096..16384 tokens, 8 kv heads (2.68 GB): 436 us = 6.15 TB/s; dealt by request and key range
// in eight rounds, with most ranges of the shorter contexts empty, 487 us.  256 of 100..4000: 378 us (461).  One of 32000:
// 31 us (53).
// kShares false: one workgroup per request and kv head.
template <bool kShares>
__global__ __launch_bounds__(kThreads, 2) void decode_attn_kernel(DecParams p) {
  __shared__ __attribute__((aligned(16))) __bf16 smem[kStages * kBN * (kKsStride + kVsStride)];
  __shared__ int wave_tiles[kWaves];
  __shared__ int seg_r, seg_t;
  __bf16* const Ks = smem;                                // [kStages][kBN][kKsStride]
  __bf16* const Vs = smem + kStages * kBN * kKsStride;    // [kStages][kBN][kVsStride]

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15;   // column of the MFMA tiles: the query head
  const int g4 = lane >> 4;    // lane group: keys 4 g4 .. 4 g4 + 3 of the wavefront's 16
  // kv head fastest: the workgroups that read the same pages (each its own 256-byte slice of every token row)
  // are dispatched together, one per XCD, and walk the pages at the same time
  const int kvh = blockIdx.x % p.Hkv;
  const int share = blockIdx.x / p.Hkv;
  const int G = p.G;
  const float c = p.scale * kLog2e;

  // ---- which tiles: `left` of them from tile t of request r on
  int r = share, t = 0, left = 0;
  if constexpr (kShares) {
    const int per = (p.n_req + kThreads - 1) / kThreads;   // requests per thread, consecutive ones
    const int r0 = min(tid * per, p.n_req), r1 = min(r0 + per, p.n_req);
    int own = 0;
    for (int i = r0; i < r1; ++i) {
      const int nt = tiles_of(p, i);
      own += nt;
      if (nt == 0 && i % p.n_shares == share) {   // an empty context: no share holds a tile of it
        u32x4* const dst = (u32x4*)((__bf16*)p.out + ((size_t)i * p.Hq + kvh * G) * kD);
        for (int k = 0; k < G * kD / 8; ++k) dst[k] = u32x4{0u, 0u, 0u, 0u};
      }
    }
    int upto = skv_wave_scan(own);
    if (lane == 63) wave_tiles[wave] = upto;
    __syncthreads();
    int total = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      const int x = wave_tiles[w];
      if (w < wave) upto += x;
      total += x;
    }
    int before = upto - own;
    const int n = min(p.n_shares, total);
    if (blockIdx.x == 0) {   // the merge kernel finds its pieces from these
      const bool by_req = p.n_cuts == p.n_req;
      if (!by_req) {
        for (int i = tid; i < p.n_cuts; i += kThreads) p.cuts[i].x = -1;
        __syncthreads();
      }
      int x = before;
      for (int i = r0; i < r1; ++i) {
        const int nt = tiles_of(p, i), i0 = nt > 0 ? share_of(x, total, n) : 0;
        const bool cut = nt > 0 && x + nt > share_begin(i0 + 1, total, n);
        if (by_req || cut) p.cuts[by_req ? i : i0] = make_int4(cut ? i : -1, x, x + nt, total);
        x += nt;
      }
    }
    if (share >= n) return;
    const int begin = share_begin(share, total, n);
    left = share_begin(share + 1, total, n) - begin;
    if (before <= begin && begin < upto) {
      int i = r0, nt = tiles_of(p, i);
      for (; before + nt <= begin; nt = tiles_of(p, i)) {
        before += nt;
        ++i;
      }
      seg_r = i;
      seg_t = begin - before;
    }
    __syncthreads();
    r = seg_r;
    t = seg_t;
  }
  for (;; ++r, t = 0) {
  r = __builtin_amdgcn_readfirstlane(r);
  int ctx = __builtin_amdgcn_readfirstlane(p.ctx_len[r]);
  ctx = max(0, min(ctx, p.max_blocks * SKV_BLOCK_TOKENS));
  const int n_tiles = (ctx + kBN - 1) / kBN;
  const int t0 = __builtin_amdgcn_readfirstlane(t);
  const int t1 = kShares ? min(n_tiles, t0 + left) : n_tiles;

  if (t0 >= t1) {  // nothing cached
    if (kShares) continue;   // (a tile is left, so a request follows)
    for (int i = tid; i < G * kD; i += kThreads)
      ((__bf16*)p.out)[((size_t)r * p.Hq + kvh * G) * kD + i] = (__bf16)0.f;
    return;
  }

  // ---- Q fragments (B operand of S^T = K Q^T): lane holds head l16, d = 32 ks + 8 g4 .. +7
  bf16x8 qf[4];
  {
    const __bf16* src = (const __bf16*)p.q + ((size_t)r * p.Hq + kvh * G + min(l16, G - 1)) * kD + 8 * g4;
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      qf[ks] = *(const bf16x8*)(src + ks * 32);
      if (l16 >= G)
#pragma unroll
        for (int e = 0; e < 8; ++e) qf[ks][e] = (__bf16)0.f;
    }
  }

  // ---- key-group addresses: lane g of window w holds where keys 16 (4 (t0 + 16 w) + g) .. + 15 start
  const unsigned row_bytes = (unsigned)p.Hkv * kD * 2u;
  auto fetch_window = [&](int w, uint64_t& ak, uint64_t& av) __attribute__((always_inline)) {
    const int gi = (t0 + 16 * w) * 4 + lane;
    uint64_t k = 0, v = 0;   // 0: no data (past the context, or a page id outside the pool), reads as zeros
    if (gi * SKV_BLOCK_TOKENS < ctx && gi < p.max_blocks) {
      const int page = p.page_table[(size_t)r * p.max_blocks + gi];
      if (page >= 0 && page < p.n_pages) {
        const uint64_t off = ((uint64_t)page * SKV_BLOCK_TOKENS * p.Hkv + kvh) * (kD * 2);
        k = (uint64_t)p.kpool + off;
        v = (uint64_t)p.vpool + off;
      }
    }
    ak = k;
    av = v;
  };
  auto lane_bcast = [&](uint64_t x, int idx) __attribute__((always_inline)) {
    const uint32_t lo = __builtin_amdgcn_readlane((int)(uint32_t)x, idx);
    const uint32_t hi = __builtin_amdgcn_readlane((int)(uint32_t)(x >> 32), idx);
    return (void*)(((uint64_t)hi << 32) | lo);
  };
  uint64_t ak_cur, av_cur, ak_nxt = 0, av_nxt = 0;
  fetch_window(0, ak_cur, av_cur);

  // ---- global -> registers -> LDS: 16 threads x 16 B per key row, four 16-key groups per tile.  Buffer
  // loads check each lane's offset against the bytes that exist from the group's base on, so the rows of
  // the last page past ctx come back as zeros, whatever the pool holds there, and so does an absent page (no bytes exist).
  u32x4 kregA[4], vregA[4], kregB[4], vregB[4];  // two tiles in flight: kt+1 (landed or landing) and kt+2
  const int t_row = tid >> 4;
  const unsigned t_off = (unsigned)t_row * row_bytes + (unsigned)(tid & 15) * 16u;
  auto load_tile = [&](int kt, u32x4 (&kreg)[4], u32x4 (&vreg)[4], uint64_t ak_w, uint64_t av_w) __attribute__((always_inline)) {
#pragma unroll
    for (int cc = 0; cc < 4; ++cc) {
      const int idx = (((kt - t0) & 15) << 2) + cc;
      int n_valid = ctx - (kt * kBN + cc * 16);  // clamped to 0..16 on the scalar unit
      asm("s_max_i32 %0, %1, 0\n\ts_min_i32 %0, %0, 16" : "=s"(n_valid) : "s"(n_valid) : "scc");
      void* const ka = lane_bcast(ak_w, idx);
      const int nrec = ka ? n_valid * (int)row_bytes : 0;
      const __amdgpu_buffer_rsrc_t rk = __builtin_amdgcn_make_buffer_rsrc(ka, 0, nrec, 0x00020000);
      const __amdgpu_buffer_rsrc_t rv = __builtin_amdgcn_make_buffer_rsrc(lane_bcast(av_w, idx), 0, nrec, 0x00020000);
      // cache policy 2 = non-temporal: every byte is used once, so the stream should not displace what L2 holds
      kreg[cc] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rk, (int)t_off, 0, 2));
      vreg[cc] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rv, (int)t_off, 0, 2));
    }
  };
  const int k_lds = t_row * kKsStride + (tid & 15) * 8;
  const int v_lds = t_row * kVsStride + (tid & 15) * 8;
  auto store_tile = [&](int kt, const u32x4 (&kreg)[4], const u32x4 (&vreg)[4]) __attribute__((always_inline)) {
    __bf16* kd = Ks + ((kt - t0) % kStages) * (kBN * kKsStride) + k_lds;
    __bf16* vd = Vs + ((kt - t0) % kStages) * (kBN * kVsStride) + v_lds;
#pragma unroll
    for (int cc = 0; cc < 4; ++cc) {
      *(u32x4*)(kd + cc * 16 * kKsStride) = kreg[cc];
      *(u32x4*)(vd + cc * 16 * kVsStride) = vreg[cc];
    }
  };

  // ---- per-wavefront softmax state over its share of the keys
  f32x4 o[8];  // O^T tiles: d = 16 a + 4 g4 + i, head = l16
#pragma unroll
  for (int a = 0; a < 8; ++a) o[a] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m_run = -INFINITY;  // running maximum of head l16 (raw score units), same in the four lane groups
  float l_run = 0.f;        // running sum over this lane group's keys

  const int k_lane = (16 * wave + l16) * kKsStride + 8 * g4;
  const int v_lane = (16 * wave + 4 * g4 + (l16 >> 2)) * kVsStride + 4 * (l16 & 3);
  auto compute = [&](int kt) __attribute__((always_inline)) {
    const __bf16* kb = Ks + ((kt - t0) % kStages) * (kBN * kKsStride) + k_lane;
    const __bf16* vb = Vs + ((kt - t0) % kStages) * (kBN * kVsStride) + v_lane;
    f32x4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < 4; ++ks)
      s = __builtin_amdgcn_mfma_f32_16x16x32_bf16(*(const bf16x8*)(kb + ks * 32), qf[ks], s, 0, 0, 0);
    // The scores are read by vector instructions right behind a branch (the ragged-tile test below).  The compiler's
    // wait-state insertion does not look through that branch, and without the states an MFMA result needs before a
    // vector instruction may read it the row maxima are taken from registers the matrix core has not written yet
    // (seen as run-to-run differences in the last bits).  Twelve idle states cover the four-pass MFMA.
    asm volatile("s_nop 7\n\ts_nop 3" : "+v"(s));
    const int key0 = kt * kBN + 16 * wave + 4 * g4;
    if (kt * kBN + kBN > ctx) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (key0 + i >= ctx) s[i] = -INFINITY;
    }
    float mx = fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3]));
    mx = skv_over_rows(mx, SkvMax());
    const float m_new = fmaxf(m_run, mx);
    float alpha = 1.f;
    f32x4 pr = {0.f, 0.f, 0.f, 0.f};
    if (m_new != -INFINITY) {
      alpha = __builtin_amdgcn_exp2f((m_run - m_new) * c);
      const float mc = m_new * c;
#pragma unroll
      for (int i = 0; i < 4; ++i) pr[i] = __builtin_amdgcn_exp2f(s[i] * c - mc);
    }
    m_run = m_new;
    l_run = l_run * alpha + ((pr[0] + pr[1]) + (pr[2] + pr[3]));
    // The weights as the sum of two bf16 values each: the matrix core idles here, and with eight bits their rounding shows in the
    // result next to its own (2-norm against 64 bits, contexts of 3000 to 32000: 2.0e-3 to 2.2e-3, now 1.63e-3 to 1.67e-3).
    s16x4 pf[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      u32x2 pw;
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        pw[j] = __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2{pr[2 * j], pr[2 * j + 1]}), bf16x2));
        pr[2 * j] -= __builtin_bit_cast(float, pw[j] << 16);
        pr[2 * j + 1] -= __builtin_bit_cast(float, pw[j] & 0xffff0000u);
      }
      pf[k] = __builtin_bit_cast(s16x4, pw);
    }
    s16x4 vf[8];
#pragma unroll
    for (int a = 0; a < 8; ++a) {
      vf[a] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(vb + 16 * a));
      o[a] = o[a] * alpha;
      o[a] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(vf[a], pf[0], o[a], 0, 0, 0);
    }
#pragma unroll
    for (int a = 0; a < 8; ++a) o[a] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(vf[a], pf[1], o[a], 0, 0, 0);
  };

  // ---- main loop: while tile kt is computed, tile kt+1 sits in one register set (on its way to LDS) and the
  // loads of tile kt+2 are in flight into the other; one barrier per tile.  Window w covers tiles
  // t0 + 16 w .. + 15; the window of tile kt+2 is fetched one iteration before that tile is requested.
  int cur_w = 0;
  auto window_of = [&](int kt, uint64_t& ak, uint64_t& av) __attribute__((always_inline)) {
    const bool nxt = ((kt - t0) >> 4) != cur_w;
    ak = nxt ? ak_nxt : ak_cur;
    av = nxt ? av_nxt : av_cur;
  };
  uint64_t akw, avw;
  load_tile(t0, kregA, vregA, ak_cur, av_cur);
  if (t0 + 1 < t1) load_tile(t0 + 1, kregB, vregB, ak_cur, av_cur);   // tile t0+1 is in window 0 (16 tiles per window)
  store_tile(t0, kregA, vregA);
  __syncthreads();
  auto step = [&](int kt, u32x4 (&k_next)[4], u32x4 (&v_next)[4], u32x4 (&k_far)[4], u32x4 (&v_far)[4]) __attribute__((always_inline)) {
    // k_next holds tile kt+1 (requested one step ago); k_far is free and takes tile kt+2
    if (((kt - t0) >> 4) != cur_w) { cur_w = (kt - t0) >> 4; ak_cur = ak_nxt; av_cur = av_nxt; }
    if (((kt - t0 + 3) & 15) == 0 && kt + 3 < t1) fetch_window((kt - t0 + 3) >> 4, ak_nxt, av_nxt);
    if (kt + 2 < t1) {
      window_of(kt + 2, akw, avw);
      load_tile(kt + 2, k_far, v_far, akw, avw);
    }
    compute(kt);
    if (kt + 1 < t1) store_tile(kt + 1, k_next, v_next);
    __syncthreads();
  };
  for (int kt = t0; kt < t1; kt += 2) {
    step(kt, kregB, vregB, kregA, vregA);
    if (kt + 1 < t1) step(kt + 1, kregA, vregA, kregB, vregB);
  }

  // ---- merge the four wavefronts' states through LDS (the tiles are no longer needed after the last barrier)
  float* red_o = (float*)smem;                       // [kWaves][16][kD]
  float* red_m = red_o + kWaves * kMaxG * kD;        // [kWaves][16]
  float* red_l = red_m + kWaves * kMaxG;
  {
    const float lt = skv_over_rows(l_run, SkvAdd());
    float* dst = red_o + (size_t)(wave * kMaxG + l16) * kD + 4 * g4;
#pragma unroll
    for (int a = 0; a < 8; ++a) *(f32x4*)(dst + 16 * a) = o[a];
    if (g4 == 0) {
      red_m[wave * kMaxG + l16] = m_run;
      red_l[wave * kMaxG + l16] = lt;
    }
  }
  __syncthreads();
  {
    const int head = tid >> 4, d0 = (tid & 15) * 8;
    if (head < G) {
      float ms = -INFINITY;
#pragma unroll
      for (int w = 0; w < kWaves; ++w) ms = fmaxf(ms, red_m[w * kMaxG + head]);
      float L = 0.f, acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int w = 0; w < kWaves; ++w) {
        const float mw = red_m[w * kMaxG + head];
        if (mw == -INFINITY) continue;
        const float wgt = __builtin_amdgcn_exp2f((mw - ms) * c);
        L += wgt * red_l[w * kMaxG + head];
        const float* src = red_o + (size_t)(w * kMaxG + head) * kD + d0;
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[j] += wgt * src[j];
      }
      if (kShares && (t0 > 0 || t1 < n_tiles)) {   // a piece of a request
        const size_t part = ((size_t)(2 * share + (t0 == 0 ? 1 : 0)) * p.Hkv + kvh) * G;
        if ((tid & 15) == 0) {
          p.part_m[part + head] = ms;
          p.part_l[part + head] = L;
        }
        float* dst = p.part_o + (part + head) * kD + d0;
#pragma unroll
        for (int j = 0; j < 8; ++j) dst[j] = acc[j];
      } else {
        const float inv = L > 0.f ? 1.f / L : 0.f;
        __bf16* dst = (__bf16*)p.out + ((size_t)r * p.Hq + kvh * G + head) * kD + d0;
#pragma unroll
        for (int j = 0; j < 8; ++j) dst[j] = (__bf16)(acc[j] * inv);
      }
    }
  }
  if (!kShares) return;
  left -= t1 - t0;
  if (left <= 0) return;
  __syncthreads();   // the merge area is read; the next request's tiles go there
  }
}

// Merge of the pieces of the requests that were cut: one workgroup per (entry of the list, query head).  Bound by latency, so no load
// waits for another: the weights of up to kThreads pieces are taken at once, one piece per thread, and the eight
// half-wavefronts then sum every eighth piece's output, 16 bytes a lane, four pieces in flight each.
__global__ __launch_bounds__(kThreads) void decode_merge_kernel(DecParams p) {
  constexpr int kTeams = kThreads / 32;
  __shared__ float wgt[kThreads], red_m[kWaves], red_l[kWaves];
  __shared__ f32x4 red_o[kTeams][32];
  const int h = blockIdx.x % p.Hq;
  const int4 cut = p.cuts[blockIdx.x / p.Hq];
  if (cut.x < 0) return;
  const int r = cut.x, tile0 = cut.y, tile1 = cut.z, total = cut.w;
  const int n = min(p.n_shares, total);
  const int i0 = share_of(tile0, total, n), i1 = share_of(tile1 - 1, total, n);
  const int pieces = i1 - i0 + 1;
  const int kvh = h / p.G, head = h % p.G;
  const int tid = threadIdx.x, team = tid >> 5, d4 = tid & 31;
  const float c = p.scale * kLog2e;
  u32x2* const dst = (u32x2*)((__bf16*)p.out + ((size_t)r * p.Hq + h) * kD + 4 * d4);
  auto piece = [&](int j) { return ((size_t)(2 * (i0 + j) + (j == 0 ? 1 : 0)) * p.Hkv + kvh) * p.G + head; };
  float m0 = -INFINITY, ms = -INFINITY;   // this thread's first piece (all of them, as a rule); the largest of all
  for (int s = tid; s < pieces; s += kThreads) {
    const float m = p.part_m[piece(s)];
    if (s == tid) m0 = m;
    ms = fmaxf(ms, m);
  }
  ms = skv_over_wave(ms, SkvMax());
  if ((tid & 63) == 0) red_m[tid >> 6] = ms;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < kWaves; ++w) ms = fmaxf(ms, red_m[w]);
  float L = 0.f;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  for (int s0 = 0; s0 < pieces; s0 += kThreads) {
    const int s = s0 + tid, n_here = min(kThreads, pieces - s0);
    float w = 0.f;
    if (s < pieces) {
      const float m = s0 == 0 ? m0 : p.part_m[piece(s)];
      if (m != -INFINITY) {   // otherwise every weight of the piece is 0
        w = __builtin_amdgcn_exp2f((m - ms) * c);
        L += w * p.part_l[piece(s)];
      }
    }
    if (s0 > 0) __syncthreads();   // the weights before are done with
    wgt[tid] = w;
    __syncthreads();
#pragma unroll 4
    for (int i = team; i < n_here; i += kTeams) acc += wgt[i] * *(const f32x4*)(p.part_o + piece(s0 + i) * kD + 4 * d4);
  }
  L = skv_over_wave(L, SkvAdd());
  if ((tid & 63) == 0) red_l[tid >> 6] = L;
  red_o[team][d4] = acc;
  __syncthreads();
  if (tid < 32) {
    L = (red_l[0] + red_l[1]) + (red_l[2] + red_l[3]);
#pragma unroll
    for (int g = 1; g < kTeams; ++g) acc += red_o[g][d4];
    const float inv = L > 0.f ? 1.f / L : 0.f;
    const bf16x2 y0 = __builtin_convertvector(f32x2{acc[0] * inv, acc[1] * inv}, bf16x2);
    const bf16x2 y1 = __builtin_convertvector(f32x2{acc[2] * inv, acc[3] * inv}, bf16x2);
    *dst = u32x2{__builtin_bit_cast(uint32_t, y0), __builtin_bit_cast(uint32_t, y1)};
  }
}

int check_decode(const skv_attn_desc* d) {
  if (!d) return SKV_EINVAL;
  if (d->dtype != SKV_BF16 || d->head_dim != kD) return SKV_EINVAL;
  if (d->n_q_heads < 1 || d->n_kv_heads < 1 || d->n_q_heads % d->n_kv_heads) return SKV_EINVAL;
  if (d->n_q_heads / d->n_kv_heads > kMaxG) return SKV_EINVAL;
  return SKV_OK;
}

// Shares per kv head: one workgroup per slot of the chip (two or four rounds: slower throughout, up to 2 x for few requests).
// 0, a workgroup per request and no merge, where contexts are so short that cutting them costs more than it gains: one
// request of 2 / 4 / 6 / 8 tiles takes 5.8 / 8.0 / 10.5 / 13.3 us whole and 9.9 us cut; 16 of 8 kv heads of 11 / 16 tiles 18.5 /
// 24.9 whole, 20.0 / 22.1 cut, and where only one of them is that long 15.6 / 17.6 cut; 64 of 8 kv heads of 11 / 16 tiles
// 34.8 / 48.0 whole, 36.9 / 50.4 cut; 128 of one kv head of 11 / 16 tiles 18.5 / 24.7 whole, 27.9 / 29.9 cut.
int64_t max_tiles_of(int32_t max_blocks) { return ((int64_t)max_blocks * SKV_BLOCK_TOKENS + kBN - 1) / kBN; }
int64_t most_shares(const skv_attn_desc* d, int32_t n_req, int32_t max_blocks) {
  return std::min<int64_t>(std::max(kSlots / d->n_kv_heads, 1), n_req * max_tiles_of(max_blocks));
}
int shares_for(const skv_attn_desc* d, int32_t n_req, int32_t max_blocks) {
  const int64_t max_tiles = max_tiles_of(max_blocks);
  const int64_t units = (int64_t)n_req * d->n_kv_heads;
  if (max_tiles <= (units < kSlots / 4 ? 5 : n_req <= 16 ? 11 : 16) || n_req * max_tiles > 0x7fffffff) return 0;
  return (int)most_shares(d, n_req, max_blocks);
}
// Room for shares whether the call takes them or not: the size never falls as n_req or max_blocks grow, so a workspace of the
// largest batch serves every smaller one.
struct Workspace {
  size_t part_m, part_l, part_o, bytes;
};
Workspace workspace_for(const skv_attn_desc* d, int32_t n_req, int32_t max_blocks) {
  const size_t shares = (size_t)most_shares(d, n_req, max_blocks), pieces = 2 * shares * d->n_q_heads;
  Workspace w;
  w.part_m = skv_align256(shares * sizeof(int4));
  w.part_l = w.part_m + skv_align256(pieces * sizeof(float));
  w.part_o = w.part_l + skv_align256(pieces * sizeof(float));
  w.bytes = std::max<size_t>(w.part_o + pieces * kD * sizeof(float), 256);
  return w;
}

}  // namespace

extern "C" int skv_decode_attn_workspace_size(const skv_attn_desc* desc, int32_t n_req, int32_t max_blocks,
                                              size_t* bytes) {
  int rc = check_decode(desc);
  if (rc) return rc;
  if (n_req < 0 || max_blocks < 0 || !bytes) return SKV_EINVAL;
  *bytes = workspace_for(desc, n_req, max_blocks).bytes;
  return SKV_OK;
}

extern "C" int skv_decode_attn(const skv_attn_desc* desc, int32_t n_req, const void* d_q, const void* d_kpool,
                               const void* d_vpool, int32_t n_pages, const int32_t* d_ctx_len,
                               const int32_t* d_page_table, int32_t max_blocks, void* d_out, void* d_workspace,
                               size_t workspace_bytes, void* stream) {
  int rc = check_decode(desc);
  if (rc) return rc;
  if (n_req < 0 || n_pages < 0 || max_blocks < 0) return SKV_EINVAL;
  if (n_req == 0) return SKV_OK;
  if (!d_q || !d_ctx_len || !d_out) return SKV_EINVAL;
  if (max_blocks > 0 && (!d_page_table || !d_kpool || !d_vpool)) return SKV_EINVAL;
  if (((uintptr_t)d_q | (uintptr_t)d_kpool | (uintptr_t)d_vpool | (uintptr_t)d_out | (uintptr_t)d_workspace) & 15)
    return SKV_EINVAL;
  size_t need = 0;
  skv_decode_attn_workspace_size(desc, n_req, max_blocks, &need);
  if (!d_workspace || workspace_bytes < need) return SKV_ENOMEM;
  const int shares = shares_for(desc, n_req, max_blocks);
  const int64_t grid = (int64_t)(shares ? shares : n_req) * desc->n_kv_heads;
  if (grid > 0x7fffffff || (int64_t)n_req * desc->n_q_heads > 0x7fffffff) return SKV_ERANGE;
  hipStream_t st = (hipStream_t)stream;
  char* ws = (char*)d_workspace;
  const Workspace w = workspace_for(desc, n_req, max_blocks);
  DecParams p;
  p.q = d_q; p.kpool = d_kpool; p.vpool = d_vpool; p.out = d_out;
  p.ctx_len = d_ctx_len; p.page_table = d_page_table;
  p.cuts = (int4*)ws;
  p.part_m = (float*)(ws + w.part_m); p.part_l = (float*)(ws + w.part_l); p.part_o = (float*)(ws + w.part_o);
  p.n_req = n_req; p.max_blocks = max_blocks; p.n_pages = n_pages;
  p.Hq = desc->n_q_heads; p.Hkv = desc->n_kv_heads; p.G = desc->n_q_heads / desc->n_kv_heads;
  p.n_shares = shares; p.scale = skv_softmax_scale(desc);
  p.n_cuts = std::min(n_req, shares - 1);
  if (shares == 0)
    decode_attn_kernel<false><<<(int)grid, kThreads, 0, st>>>(p);
  else
    decode_attn_kernel<true><<<(int)grid, kThreads, 0, st>>>(p);
  SKV_HIP(hipGetLastError());
  if (shares > 1) {
    decode_merge_kernel<<<p.n_cuts * desc->n_q_heads, kThreads, 0, st>>>(p);
    SKV_HIP(hipGetLastError());
  }
  return SKV_OK;
}
