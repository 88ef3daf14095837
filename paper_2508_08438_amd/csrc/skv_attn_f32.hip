// Causal GQA prefill attention, fp32: the same result as the bf16 path (SafeKV Section 2.1 over the reused prefix and
// the request's own new rows), with fp32 accuracy in products, sums and softmax.
//
// The contractions run on the bf16 matrix instruction, whose rate is sixteen times that of the fp32 one, on operands split
// into three bf16 pieces each (exactly; what has no exact pieces is taken row by row in plain fp32): a = a0 + a1 + a2, a . b =
// the six products a_i b_j with i + j <= 2, all accumulated in fp32; what is left out is below 2^-24 of the product.  Against
// 64-bit sums the results are 1.1e-7 to 2.2e-7 off (2-norm; N(0,1) inputs, 200 to 3000 keys) where fp32 multiply-adds, one key
// after another per lane, are 1.7e-7 to 2.9e-7 off and the fp32 matrix instruction 2.3e-7 to 5.8e-7; with scores 6 and 30
// times as wide the three keep that order.  The products are formed transposed, S^T = K Q^T and O^T = V^T P^T, so a query is a
// lane column: the softmax is a register reduction plus one exchange between the halves of the wavefront, and the accumulator
// registers of S^T are the B operand of the second product as they stand.
#include <algorithm>
#include <type_traits>

#include "skv_gather.h"

namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kRows = 32;       // query rows per wavefront
constexpr int kWaves = 4;
constexpr int kThreads = 64 * kWaves;
constexpr int kKeys = 32;       // keys per step of a wavefront
constexpr int kPieces = 3;
constexpr float kLog2e = 1.4426950408889634f;

// A float as the sum of three bf16 values: its 24 significant bits in pieces of eight.  Each piece is the rounding of what the
// pieces before leave, so nothing is lost (the differences are exact) as long as the last piece is a normal number.
struct Pieces {
  bf16x8 p[kPieces];
};
__device__ __forceinline__ Pieces split8(const float (&x)[8]) {
  u32x4 w[kPieces];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    float a = x[2 * i], b = x[2 * i + 1];
#pragma unroll
    for (int k = 0; k < kPieces; ++k) {
      const uint32_t h = __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2{a, b}), bf16x2));
      w[k][i] = h;
      if (k + 1 < kPieces) {
        a -= __builtin_bit_cast(float, h << 16);
        b -= __builtin_bit_cast(float, h & 0xffff0000u);
      }
    }
  }
  Pieces r;
#pragma unroll
  for (int k = 0; k < kPieces; ++k) r.p[k] = __builtin_bit_cast(bf16x8, w[k]);
  return r;
}
// The same in 16 steps of 16 values (8 of 8): a pair's first piece and what it leaves, then the other two.
typedef u32x4 Words[kPieces];
__device__ __forceinline__ void split_step(float& a, float& b, bool second, int at, Words& w) {
  auto piece = [&](int k) __attribute__((always_inline)) {
    const uint32_t h = __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2{a, b}), bf16x2));
    w[k][at] = h;
    if (k == 2) return;
    a -= __builtin_bit_cast(float, h << 16);
    b -= __builtin_bit_cast(float, h & 0xffff0000u);
  };
  if (!second) {
    piece(0);
  } else {
    piece(1);
    piece(2);
  }
}
// Products of pieces i + j = kSum, added to acc.  A sum that takes the small ones first, or apart, is rounded at its full size
// by the products of the first pieces only: that is what makes it as exact as a chain of fp32 multiply-adds.
template <int kSum>
__device__ __forceinline__ f32x16 mfma_pieces(const Pieces& a, const Pieces& b, f32x16 acc) {
#pragma unroll
  for (int i = 0; i <= kSum; ++i) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.p[i], b.p[kSum - i], acc, 0, 0, 0);
  return acc;
}

// op over a value and the one 32 lanes away
template <typename Op>
__device__ __forceinline__ float over_halves(float x, Op op) {
  float a = x, b = x;
  skv_swap_halves(a, b);
  return op(a, b);
}

template <int N> struct vec_of;
template <> struct vec_of<2> { typedef f32x2 type; };
template <> struct vec_of<4> { typedef f32x4 type; };

// ---- which work item: (request, row tile, query head).  Request r's tiles start at q_off[r] / tile_rows + r: at least
// ceil(S_r / tile_rows) apart, so every tile has a place and the place is found from q_off alone (64 requests per step); places
// no tile maps to leave at once.
struct Item {
  int h, hk, r, qbase, S, L, row0, row1;
  // Request lane's rows from what q_off is made of, for up to 64 requests: their end (the launch that writes q_off need not come first).
  static __device__ __forceinline__ int rows_end(const SkvAttnF32Params& p, int& own) {
    const int lane = threadIdx.x & 63;
    own = lane < p.n_req ? max(0, p.req_off[lane + 1] - p.req_off[lane] - p.matched_len[lane]) : 0;
    return skv_wave_scan(own);
  }
  // kStep: q_off is being written by the same launch.  (Known at compile time: asked in every workgroup it cost each call 0.2 to 0.3 us; one row behind
  // 16 keys 5.92 -> 5.71.)
  template <int kTileRows, bool kStep>
  __device__ __forceinline__ bool find(const SkvAttnF32Params& p, int block) {
    const int lane = threadIdx.x & 63;
    h = block % p.Hq;
    hk = h / (p.Hq / p.Hkv);
    const int t = block / p.Hq;
    r = 0;
    if constexpr (kStep) {
      int own;
      const int end = rows_end(p, own);
      r = __builtin_popcountll(__ballot(lane < p.n_req && (end - own) / kTileRows + lane <= t)) - 1;   // (lane 0 always counts)
      qbase = __builtin_amdgcn_readlane(end - own, r);
      S = __builtin_amdgcn_readlane(own, r);
    } else {
      for (int n = p.n_req; n > 1;) {
        const int step = (n + 63) / 64;
        const int idx = r + lane * step;
        const bool before = idx < r + n && p.q_off[idx] / kTileRows + idx <= t;
        const int k = __builtin_popcountll(__ballot(before));   // lane 0 always counts (t is at or behind the first place)
        const int lo = r + (k > 0 ? k - 1 : 0) * step;
        n = min(step, r + n - lo);
        r = lo;
      }
      r = __builtin_amdgcn_readfirstlane(r);
      qbase = __builtin_amdgcn_readfirstlane(p.q_off[r]);
      S = __builtin_amdgcn_readfirstlane(p.q_off[r + 1]) - qbase;
    }
    S = (int)min((int64_t)S, p.max_rows - qbase);
    const int n_tiles = (S + kTileRows - 1) / kTileRows;
    const int k_tile = t - (qbase / kTileRows + r);
    if (k_tile < 0 || k_tile >= n_tiles) return false;
    L = __builtin_amdgcn_readfirstlane(p.matched_len[r]);
    L = L > 0 ? L & ~(SKV_BLOCK_TOKENS - 1) : 0;               // whole blocks only
    row0 = (n_tiles - 1 - k_tile) * kTileRows;                 // the request's heaviest tile first
    row1 = min(S, row0 + kTileRows);
    return true;
  }
  // The same places, dealt out anew among each 64 requests: of all of them the last tiles come first, by their number in the request (64
  // requests of 1070 rows over 512 places: the chip empties 1 % after the mean and not 11 %).  What a request's rows leave over is its
  // first tile, which sees the fewest keys, and so many rows more that a wavefront's start where a block of keys does.
  template <int kTileRows, bool kStep>
  __device__ __forceinline__ bool find_by_number(const SkvAttnF32Params& p, int block) {
    const int lane = threadIdx.x & 63;
    h = block % p.Hq;
    hk = h / (p.Hq / p.Hkv);
    const int t = block / p.Hq;
    int r0 = 0;   // first of the 64 (a step has no more)
    for (int n = kStep ? 1 : (p.n_req + 63) / 64; n > 1;) {
      const int step = (n + 63) / 64, idx = lane * step;
      const bool before = idx < n && p.q_off[r0 + 64 * idx] / kTileRows + r0 + 64 * idx <= t;
      const int k = __builtin_popcountll(__ballot(before));
      const int lo = (k > 0 ? k - 1 : 0) * step;
      n = min(step, n - lo);
      r0 += 64 * lo;
    }
    r0 = __builtin_amdgcn_readfirstlane(r0);
    const bool have = r0 + lane < p.n_req;
    int begin = 0, rows = 0;
    if constexpr (kStep) {
      const int end = rows_end(p, rows);
      begin = end - rows;
    } else if (have) {
      begin = p.q_off[r0 + lane];
      rows = p.q_off[r0 + lane + 1] - begin;
    }
    rows = (int)min((int64_t)rows, p.max_rows - begin);
    const int own = have ? max(0, (rows + kTileRows - 1) / kTileRows) : 0;
    int place = t - (__builtin_amdgcn_readfirstlane(begin) / kTileRows + r0);
    auto from = [&](int number) __attribute__((always_inline)) { return skv_over_wave(max(0, own - number), SkvAdd()); };   // tiles of that number and higher ones
    int lo = 0, hi = skv_over_wave(own, SkvMax());
    if (place < 0 || place >= from(0)) return false;
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (from(mid) > place) lo = mid; else hi = mid;
    }
    const int tile = __builtin_amdgcn_readfirstlane(lo);
    place -= __builtin_amdgcn_readfirstlane(from(tile + 1));
    const uint64_t with = __ballot(own > tile);
    const int at = __builtin_ctzll(__ballot(own > tile && __builtin_popcountll(with & ((1ull << lane) - 1)) == place));
    r = r0 + at;
    qbase = __builtin_amdgcn_readlane(begin, at);
    S = __builtin_amdgcn_readlane(rows, at);
    L = __builtin_amdgcn_readfirstlane(p.matched_len[r]);
    L = L > 0 ? L & ~(SKV_BLOCK_TOKENS - 1) : 0;               // whole blocks only
    int first = S - (__builtin_amdgcn_readlane(own, at) - 1) * kTileRows;
    const int more = -(L + first) & (kKeys - 1);
    if (first + more <= kTileRows) first += more;
    row0 = tile > 0 ? first + (tile - 1) * kTileRows : 0;
    row1 = min(S, first + tile * kTileRows);
    return true;
  }
};

// ---- rows in plain fp32 arithmetic: a wavefront per row and head.  A lane takes every 64th key with a softmax state
// and an output of its own; in the end the lanes' outputs are summed so that each is left with every 64th value.
struct Row {
  int r, L, qbase, tok, h;   // request, its reused length, its first row in Q, the row, the head
};
// kKept: values of the output kept at once; with fewer than D the keys are scored again for the next.
template <int D, int kKept>
__device__ __forceinline__ void one_row(const SkvAttnF32Params& p, const Row& row) {
  const int lane = threadIdx.x & 63, hk = row.h / (p.Hq / p.Hkv);
  const int n_keys = row.L + row.tok - row.qbase + 1;
  constexpr int kLoad = 64;   // values of a K or V row in flight; of 128, K and V at once would not fit the registers
  const float c = p.scale * kLog2e;
  // (one row for the whole wavefront: through the scalar unit, no vector registers)
  const auto q = (const __attribute__((address_space(4))) float*)((uint64_t)p.q + ((uint64_t)row.tok * p.Hq + row.h) * (D * 4));
#pragma unroll 1
  for (int first = 0; first < D; first += kKept) {
  float m = -INFINITY, l = 0.f, acc[kKept];
#pragma unroll
  for (int d = 0; d < kKept; ++d) acc[d] = 0.f;
  for (int key = lane; key < n_keys; key += 64) {
    const float *kr = nullptr, *vr = nullptr;   // an absent page reads as zeros
    if (key < row.L) {
      const int g = key / SKV_BLOCK_TOKENS, page = g < p.max_blocks ? p.page_table[(size_t)row.r * p.max_blocks + g] : -1;
      if (page >= 0 && page < p.n_pages) {
        const size_t off = (((size_t)page * SKV_BLOCK_TOKENS + key % SKV_BLOCK_TOKENS) * p.Hkv + hk) * D;
        kr = (const float*)p.kpool + off;
        vr = (const float*)p.vpool + off;
      }
    } else {
      const size_t off = ((size_t)(row.qbase + key - row.L) * p.Hkv + hk) * D;
      kr = (const float*)p.knew + off;
      vr = (const float*)p.vnew + off;
    }
    float s = 0.f;
    if (kr) {
      f32x4 sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int d0 = 0; d0 < D; d0 += kLoad) {
        f32x4 x[kLoad / 4];
#pragma unroll
        for (int i = 0; i < kLoad / 4; ++i) x[i] = *(const f32x4*)(kr + d0 + 4 * i);
#pragma unroll
        for (int d = 0; d < kLoad; ++d) sum[d % 4] = __builtin_fmaf(q[d0 + d], x[d / 4][d % 4], sum[d % 4]);
        if (D > 64) __builtin_amdgcn_sched_barrier(0);
      }
      s = ((sum[0] + sum[1]) + (sum[2] + sum[3])) * c;
    }
    const float m_new = fmaxf(m, s), ref = m_new == -INFINITY ? 0.f : m_new;
    const float alpha = __builtin_amdgcn_exp2f(m - ref), w = __builtin_amdgcn_exp2f(s - ref);
    m = m_new;
    l = l * alpha + w;
    if (vr) {
#pragma unroll
      for (int d0 = 0; d0 < kKept; d0 += kLoad) {
        f32x4 x[kLoad / 4];
#pragma unroll
        for (int i = 0; i < kLoad / 4; ++i) x[i] = *(const f32x4*)(vr + first + d0 + 4 * i);
#pragma unroll
        for (int d = 0; d < kLoad; ++d) acc[d0 + d] = acc[d0 + d] * alpha + w * x[d / 4][d % 4];
        if (D > 64) __builtin_amdgcn_sched_barrier(0);
      }
    } else {
#pragma unroll
      for (int d = 0; d < kKept; ++d) acc[d] *= alpha;
    }
  }
  const float all = skv_over_wave(m, SkvMax());
  const float f = __builtin_amdgcn_exp2f(m - (all == -INFINITY ? 0.f : all));   // a lane without a key: 0
  l *= f;
  l = skv_over_wave(l, SkvAdd());
  float* const out = (float*)p.out + ((size_t)row.tok * p.Hq + row.h) * D + first + lane;
#pragma unroll
  for (int v = 0; v < kKept / 64; ++v) {
    float a[64];
#pragma unroll
    for (int d = 0; d < 64; ++d) a[d] = acc[64 * v + d] * f;
#pragma unroll
    for (int n = 32; n >= 1; n >>= 1)   // the halves of the wavefront swap halves of what is left: lane i ends with value i
#pragma unroll
      for (int d = 0; d < n; ++d) {
        const bool up = lane & n;
        const float keep = up ? a[d + n] : a[d], give = up ? a[d] : a[d + n];
        a[d] = keep + __shfl_xor(give, n);
      }
    out[64 * v] = a[0] / l;
  }
  }
}

// What has no exact pieces: infinities and NaN, which a matrix product would also carry into rows that do not see their key,
// values that round to infinity as bf16, and magnitudes so small that a piece would not be a normal number.  A tile that met one
// is taken again row by row, over the keys the row sees.
template <int D, int W>
__device__ __forceinline__ void rows_one_by_one(const SkvAttnF32Params& p, const Item& it) {
  for (int i = it.row0 + (threadIdx.x >> 6); i < it.row1; i += W) {
    const Row row = {it.r, it.L, it.qbase, __builtin_amdgcn_readfirstlane(it.qbase + i), it.h};
    one_row<D, 64>(p, row);   // (all 128 at once would cost the tile's loop registers)
  }
}
// Small magnitudes.  Pieces are exact down to 2^-110.  Q within [2^-100, 2^80] (or zero) splits exactly, and what K's pieces lose,
// 2^-134 at the most, then changes a score by less than 2^-47; a column of V with a value of 2^-95 or more loses less than 2^-39
// of it.  The weights need no such rule: what they lose is 2^-134 of a row's largest.
struct RangeOfQ {
  uint32_t least = 0xffffffffu, most = 0;   // of the magnitudes' bits, less one (so that zero does not count), and as they are
  __device__ __forceinline__ void add(float x) {
    const uint32_t u = __builtin_bit_cast(uint32_t, x) & 0x7fffffffu;
    least = min(least, u - 1u);
    most = max(most, u);
  }
  __device__ __forceinline__ bool odd() const { return least < ((127u - 100u) << 23) - 1u || most > (127u + 80u) << 23; }
};
// Where a sum over a column is that small, its values need a look (tiny_columns): of values (or zeros) below 2^-95 any is, up to 2^23 keys, whose weights are 4 on
// average at the most (kSumLimit of a lane's 16).
template <int kA>
__device__ __forceinline__ bool some_small(const f32x16 (&o)[kA], float l) {
  bool small = false;
#pragma unroll
  for (int a = 0; a < kA; ++a)
#pragma unroll
    for (int e = 0; e < 16; ++e) small |= fabsf(o[a][e]) < 0x1p-70f;
  return small && l > 0.f;   // (no key, no sum)
}
// Which of the two it is: every wavefront looks at every W-th 16-key group, a lane at a column.
template <int D, int W>
__device__ __forceinline__ bool tiny_columns(const SkvAttnF32Params& p, const Item& it) {
  constexpr int kPer = D / 64;
  const int lane = threadIdx.x & 63, key_end = it.L + it.row1;
  uint32_t bits[kPer] = {};
  for (int g = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); g * SKV_BLOCK_TOKENS < key_end; g += W) {
    const int key0 = g * SKV_BLOCK_TOKENS;
    const float* v = nullptr;
    if (key0 >= it.L) {
      v = (const float*)p.vnew + ((size_t)(it.qbase + key0 - it.L) * p.Hkv + it.hk) * D;
    } else if (g < p.max_blocks) {
      const int page = p.page_table[(size_t)it.r * p.max_blocks + g];
      if (page >= 0 && page < p.n_pages) v = (const float*)p.vpool + ((size_t)page * SKV_BLOCK_TOKENS * p.Hkv + it.hk) * D;
    }
    if (!v) continue;
    const int last = min(SKV_BLOCK_TOKENS, key_end - key0) - 1;
#pragma unroll
    for (int i = 0; i < SKV_BLOCK_TOKENS; ++i)
#pragma unroll
      for (int k = 0; k < kPer; ++k) bits[k] |= __builtin_bit_cast(uint32_t, v[(size_t)min(i, last) * p.Hkv * D + 64 * k + lane]);
  }
  bool tiny = false;   // no value with one of the three highest exponent bits, and not all zero
#pragma unroll
  for (int k = 0; k < kPer; ++k) tiny |= (bits[k] & 0x7fffffffu) != 0 && (bits[k] & 0x70000000u) == 0;
  return tiny;
}
template <int kA>
__device__ __forceinline__ bool all_finite(const f32x16 (&o)[kA], float l) {
#pragma unroll
  for (int a = 0; a < kA; ++a)
#pragma unroll
    for (int e = 0; e < 16; ++e) l = __builtin_fmaf(o[a][e], 0.f, l);
  return l < INFINITY;
}

// A weight is taken against the reference as it stands: that moves to the largest score so far only where a lane's weights of one block
// sum to more than kSumLimit (some score two or more above it; infinities and NaN too), or where there is none yet.  A maximum that moved with every block took 50
// of its 400 vector instructions.  The score's small products are added last, to a sum no larger than the exponent itself: the results are
// closer to 64 bits than with the maximum (2-norm, 64 requests of 1070 rows, N(0,1): 1.62e-7 -> 1.53e-7, scores 4 times as wide
// 3.24e-7 -> 2.89e-7, 30 times 7.7e-7 -> 6.6e-7; one of 250 rows 1.31e-7 -> 1.23e-7).
constexpr float kSumLimit = 64.f;
__device__ __forceinline__ float weight(float s, float s_low, float c, float ref) {
  return __builtin_amdgcn_exp2f(__builtin_fmaf(s_low, c, __builtin_fmaf(s, c, -ref)));
}
__device__ __forceinline__ float largest(const f32x16& s, const f32x16& s_low) {
  float mx = s[0] + s_low[0];
#pragma unroll
  for (int e = 1; e < 16; ++e) mx = fmaxf(mx, s[e] + s_low[e]);
  return mx;
}
// The reference of the queries whose weights summed to too much (trip; in either half), and the new weights.  Returns what everything that was
// summed against the old one is to be multiplied by.  m_ref: reference (scaled, exp2 units), l_run: this half's running sum, per query.
__device__ __forceinline__ float move_reference(const f32x16& s, const f32x16& s_low, bool trip, float c, float (&w)[16], float (&sum)[2], float& m_ref,
                                                float& l_run) {
  const float m_new = fmaxf(m_ref, over_halves(trip ? largest(s, s_low) : -INFINITY, SkvMax()) * c);
  const float ref = m_new == -INFINITY ? 0.f : m_new;
  const float alpha = __builtin_amdgcn_exp2f(m_ref - ref);
  l_run *= alpha;
  m_ref = m_new;
  sum[0] = sum[1] = 0.f;
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    w[e] = weight(s[e], s_low[e], c, ref);
    sum[e & 1] += w[e];
  }
  return alpha;
}
// `seen`: the last key the tile's first row sees
__device__ __forceinline__ void mask(f32x16& s, f32x16& s_low, int key0, int seen) {
  const int lane = threadIdx.x & 63, l32 = lane & 31, half = lane >> 5;
  if (key0 + kKeys - 1 > seen) {
    const int limit = seen + l32 - key0 - 4 * half;
#pragma unroll
    for (int e = 0; e < 16; ++e)
      if ((e >> 2) * 8 + (e & 3) > limit) {
        s[e] = -INFINITY;
        s_low[e] = 0.f;
      }
  }
}
// Scores -> weights, in place of s
template <int kA>
__device__ __forceinline__ void softmax_step(f32x16& s, f32x16& s_low, int key0, int seen, float c, f32x16 (&o)[kA], float& m_ref, float& l_run) {
  mask(s, s_low, key0, seen);
  float w[16], sum[2] = {0.f, 0.f};
  const bool none = m_ref == -INFINITY;   // no key so far, nothing summed
  if (__any(none)) m_ref = fmaxf(m_ref, over_halves(none ? largest(s, s_low) : -INFINITY, SkvMax()) * c);
  const float ref = m_ref == -INFINITY ? 0.f : m_ref;   // still none: every term is 0
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    w[e] = weight(s[e], s_low[e], c, ref);
    sum[e & 1] += w[e];
  }
  const bool trip = !(sum[0] + sum[1] <= kSumLimit);
  if (__builtin_expect(__any(trip), 0)) {
    const float alpha = move_reference(s, s_low, trip, c, w, sum, m_ref, l_run);
#pragma unroll
    for (int a = 0; a < kA; ++a)
#pragma unroll
      for (int e = 0; e < 16; ++e) o[a][e] *= alpha;
  }
  l_run += sum[0] + sum[1];
#pragma unroll
  for (int e = 0; e < 16; ++e) s[e] = w[e];
}
// the weights of a block as B operands: 16-key group g of it
__device__ __forceinline__ Pieces weights(const f32x16& s, int g) {
  float x[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) x[i] = s[8 * g + i];
  return split8(x);
}
// o += V^T P^T of one block: summed from zero, small products first, and added once
__device__ __forceinline__ void add_block(f32x16& o, const Pieces& v0, const Pieces& v1, const Pieces (&w)[2]) {
  const f32x16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  f32x16 add = mfma_pieces<2>(v0, w[0], zero16);
  add = mfma_pieces<2>(v1, w[1], add);
  add = mfma_pieces<1>(v0, w[0], add);
  add = mfma_pieces<1>(v1, w[1], add);
  add = mfma_pieces<0>(v0, w[0], add);
  add = mfma_pieces<0>(v1, w[1], add);
#pragma unroll
  for (int e = 0; e < 16; ++e) o[e] += add[e];
}

// ---- short suffixes and small batches ---------------------------------------------------------------
// One workgroup per 32 rows, whose four wavefronts take every fourth 32-key block and merge their partial softmax states
// through LDS: a small batch gets four times the wavefronts.  Every wavefront splits the keys it reads (nobody shares
// them), straight from L2 in the operand layout; only Q's pieces lie in LDS.
//   S^T: A = K, lane (key l32, half) takes d = 8 j + 4 half .. + 3 as one 16-byte load per j; two of them are the operand of
//        a step, whose slots stand for the same d in Q.
//   O^T: register e of S^T holds key 8 (e / 4) + 4 half + e % 4; A = V^T: lane (l32, half) takes the D / 32 elements
//        d = (D / 32) l32 .. of that key's row in one load; element a belongs to accumulator a, whose row m then stands for
//        d = (D / 32) m + a.
// Bound by latency and the splitting (5.5 vector instructions per value, 80 values per lane and block at D = 64).
// D = 128 has a SIMD's registers to one wavefront (two spill: 2.70 ms instead of 2.38 for 40 requests of up to 2500 rows).
// W: wavefronts of a workgroup, one where the batch fills the chip by itself (the rule stands at the end).
// Attention alone, us, on the fp32 matrix instruction -> so, four wavefronts: 8 requests of 144..320 rows, 8/8 heads, d 64: 27 -> 21; 100 of up
// to 30 rows behind 512..2048 cached ones: 140 -> 95; the same at 8/2 heads, d 128: 225 -> 227.
template <int D, int W, bool kStep>
__device__ __forceinline__ void attn_f32_item(const SkvAttnF32Params& p, int block) {
  constexpr int kWaves = W, kThreads = 64 * W;
  constexpr int kJ = D / 8;        // 16-byte pieces of a K row per lane
  constexpr int kA = D / 32;       // output accumulators
  typedef typename vec_of<kA>::type vvec;
  constexpr int kRedStride = D + kA;   // floats per query row of a partial state in LDS
  constexpr int kT = D / 16;       // steps of the score product
  constexpr int kRed = kWaves * kRows * kRedStride, kQ = 3 * kRows * D / 2;
  __shared__ __attribute__((aligned(16))) float smem[kRed > kQ ? kRed : kQ];
  u32x4* const q_lds = (u32x4*)smem;    // the pieces of Q while the loop runs: [piece][step][half][row], 8 values each,
  float* const red_o = smem;    // the partial outputs after it
  __shared__ float red_m[kWaves][kRows], red_l[kWaves][kRows];

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l32 = lane & 31, half = lane >> 5;

  Item it;
  if (!it.find<kRows, kStep>(p, block)) return;
  const int h = it.h, hk = it.hk, r = it.r, qbase = it.qbase, S = it.S, L = it.L, row0 = it.row0, row1 = it.row1;
  const int key_end = L + row1;                               // keys [0, key_end) are seen by some row of the tile
  const int n_blocks = (key_end + kKeys - 1) / kKeys;
  const float c = p.scale * kLog2e;

  // ---- where the keys of a block lie.  Lane l32 (both halves) finds the row of key 32 b + l32; a 16-key group is one pool
  // page or 16 consecutive new rows, so the V rows follow from the addresses of lanes 0 and 16.
  const uint64_t kpool_a = (uint64_t)p.kpool, vpool_a = (uint64_t)p.vpool, knew_a = (uint64_t)p.knew, vnew_a = (uint64_t)p.vnew, q_a = (uint64_t)p.q;
  const unsigned row_bytes = (unsigned)p.Hkv * D * 4u;
  auto page_of = [&](int b) __attribute__((always_inline)) {
    const int g = min(b * kKeys + l32, key_end - 1) / SKV_BLOCK_TOKENS;
    int page = -1;
    if (g * SKV_BLOCK_TOKENS < L && g < p.max_blocks) page = p.page_table[(size_t)r * p.max_blocks + g];
    return page;
  };
  auto locate = [&](int b, int page, uint64_t& ka, uint64_t& va, bool& ok) __attribute__((always_inline)) {
    const int key = min(b * kKeys + l32, key_end - 1);
    ok = true;
    if (key < L) {
      ok = page >= 0 && page < p.n_pages;
      const uint64_t off = (((uint64_t)(ok ? page : 0) * SKV_BLOCK_TOKENS + key % SKV_BLOCK_TOKENS) * p.Hkv + hk) * (D * 4);
      ka = kpool_a + off;
      va = vpool_a + off;
      if (!ok) ka = va = q_a;        // reads as zeros: any readable row will do, the loads are cleared below
    } else {
      const uint64_t off = ((uint64_t)(qbase + key - L) * p.Hkv + hk) * (D * 4);
      ka = knew_a + off;
      va = vnew_a + off;
    }
  };
  auto bcast = [&](uint64_t x, int from) __attribute__((always_inline)) {
    const uint32_t lo = __builtin_amdgcn_readlane((int)(uint32_t)x, from), hi = __builtin_amdgcn_readlane((int)(uint32_t)(x >> 32), from);
    return (const __attribute__((address_space(1))) char*)(((uint64_t)hi << 32) | lo);
  };

  f32x4 kf[kJ];
  vvec vf[16];
  f32x16 o[kA];
#pragma unroll
    for (int a = 0; a < kA; ++a)
#pragma unroll
      for (int e = 0; e < 16; ++e) o[a][e] = 0.f;
  auto load_k = [&](uint64_t ka, bool ok) __attribute__((always_inline)) {
    const auto src = (const __attribute__((address_space(1))) char*)(ka + (uint64_t)(16 * half));
#pragma unroll
    for (int j = 0; j < kJ; ++j) kf[j] = *(const __attribute__((address_space(1))) f32x4*)(src + 32 * j);
    if (__builtin_expect(!__all(ok), 0)) {
#pragma unroll
      for (int j = 0; j < kJ; ++j)
        if (!ok) kf[j] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
  };
  unsigned voff[8];   // where in a 16-key group this lane's pieces lie
#pragma unroll
  for (int e = 0; e < 8; ++e) voff[e] = (unsigned)((e >> 2) * 8 + 4 * half + (e & 3)) * row_bytes + l32 * (kA * 4);
  auto load_v = [&](int b, uint64_t va, bool ok) __attribute__((always_inline)) {
    const uint64_t good = __ballot(ok);
#pragma unroll
    for (int g = 0; g < 2; ++g) {
      const auto base = bcast(va, 16 * g);
      const bool present = (good >> (16 * g)) & 1;
      const int n_rows = present ? key_end - (b * kKeys + 16 * g) : 1;
      if (__builtin_expect(n_rows >= 16, 1)) {
#pragma unroll
        for (int e = 0; e < 8; ++e) vf[8 * g + e] = *(const __attribute__((address_space(1))) vvec*)(base + voff[e]);
      } else {   // rows past the tile's last key re-read it
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const int row = min((e >> 2) * 8 + 4 * half + (e & 3), max(n_rows, 1) - 1);
          vf[8 * g + e] = *(const __attribute__((address_space(1))) vvec*)(base + (row * row_bytes + l32 * (kA * 4)));
        }
      }
      if (__builtin_expect(!present, 0)) {
#pragma unroll
        for (int e = 0; e < 8; ++e) vf[8 * g + e] = vvec{};
      }
    }
  };

  float m_run = -INFINITY, l_run = 0.f;   // running maximum (scaled, exp2 units) and this half's running sum, per query
  const f32x16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  RangeOfQ q_range;
  int b = wave, page_nxt = -1;
  uint64_t ka = 0, va = 0;
  bool ok = true;
  if (b < n_blocks) {   // the first K rows travel while Q does
    locate(b, page_of(b), ka, va, ok);
    if (b + kWaves < n_blocks) page_nxt = page_of(b + kWaves);
    load_k(ka, ok);
  }
  // Q: through LDS, read as B operands from there (its registers would cost the second wavefront of the SIMD)
  for (int i = threadIdx.x; i < kRows * (D / 8); i += kThreads) {
    const int row = i % kRows, th = i / kRows;   // th = 2 step + half
    const f32x4* src = (const f32x4*)((const float*)p.q + ((size_t)(qbase + min(row0 + row, S - 1)) * p.Hq + h) * D + 16 * (th >> 1) + 4 * (th & 1));
    const f32x4 x0 = src[0], x1 = src[2];
    const float x[8] = {x0[0], x0[1], x0[2], x0[3], x1[0], x1[1], x1[2], x1[3]};
#pragma unroll
    for (int k = 0; k < 8; ++k) q_range.add(x[k]);
    const Pieces q = split8(x);
#pragma unroll
    for (int k = 0; k < 3; ++k) q_lds[(k * (D / 8) + th) * kRows + row] = __builtin_bit_cast(u32x4, q.p[k]);
  }
  __syncthreads();
  if (b < n_blocks) {
    // One block: its V rows travel during the scores, the next block's K rows during the softmax and the output update.
    for (; b < n_blocks; b += kWaves) {
      load_v(b, va, ok);
      __builtin_amdgcn_sched_barrier(0);
      f32x16 s = zero16, s_low = zero16;
#pragma unroll
      for (int t = 0; t < kT; ++t) {
        const f32x4 x0 = kf[2 * t], x1 = kf[2 * t + 1];
        const float x[8] = {x0[0], x0[1], x0[2], x0[3], x1[0], x1[1], x1[2], x1[3]};
        Pieces q;
#pragma unroll
        for (int i = 0; i < kPieces; ++i) q.p[i] = __builtin_bit_cast(bf16x8, q_lds[(i * (D / 8) + 2 * t + half) * kRows + l32]);
        const Pieces k = split8(x);
        s_low = mfma_pieces<2>(k, q, s_low);
        s_low = mfma_pieces<1>(k, q, s_low);
        s = mfma_pieces<0>(k, q, s);
      }
      __builtin_amdgcn_sched_barrier(0);
      if (b + kWaves < n_blocks) {
        locate(b + kWaves, page_nxt, ka, va, ok);
        load_k(ka, ok);
        if (b + 2 * kWaves < n_blocks) page_nxt = page_of(b + 2 * kWaves);
      }
      // idle states for the last score instructions: their readers may sit behind a branch, through which the compiler does
      // not count them
      asm volatile("s_nop 7\n\ts_nop 3" : "+v"(s), "+v"(s_low));
      softmax_step(s, s_low, b * kKeys, L + row0, c, o, m_run, l_run);
      __builtin_amdgcn_sched_barrier(0);
      const Pieces w[2] = {weights(s, 0), weights(s, 1)};
#pragma unroll
      for (int a = 0; a < kA; ++a) {
        Pieces v[2];
#pragma unroll
        for (int g = 0; g < 2; ++g) {
          float x[8];
#pragma unroll
          for (int i = 0; i < 8; ++i) x[i] = vf[8 * g + i][a];
          v[g] = split8(x);
        }
        add_block(o[a], v[0], v[1], w);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    asm volatile("s_nop 7\n\ts_nop 3");
  }
  l_run = over_halves(l_run, SkvAdd());
  const bool no_pieces = q_range.odd() || !all_finite(o, l_run), small = some_small(o, l_run);
  if (__builtin_expect(__syncthreads_or(no_pieces || small), 0)) {   // (Q is no longer needed behind this either)
    if (__syncthreads_or(no_pieces || tiny_columns<D, W>(p, it))) {
      rows_one_by_one<D, W>(p, it);
      return;
    }
  }

  // ---- output.  Lane (query l32, half), accumulator row e: d = kA m .. with m = 8 (e / 4) + 4 half + e % 4
  const size_t out_row = ((size_t)qbase + row0) * p.Hq + h;   // row of the workgroup's first query
  const int n_rows = row1 - row0;
  {
    float* dst = red_o + (size_t)(wave * kRows + l32) * kRedStride;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      vvec x;
#pragma unroll
      for (int a = 0; a < kA; ++a) x[a] = o[a][e];
      *(vvec*)(dst + kA * ((e >> 2) * 8 + 4 * half + (e & 3))) = x;
    }
    if (half == 0) {
      red_m[wave][l32] = m_run;
      red_l[wave][l32] = l_run;
    }
  }
  __syncthreads();
  for (int i = threadIdx.x; i < n_rows * (D / kA); i += kThreads) {
    const int row = i / (D / kA), d = (i % (D / kA)) * kA;
    float m = -INFINITY;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) m = fmaxf(m, red_m[w][row]);
    // More states are more roundings: those of eight wavefronts are summed in 64 bits, without which their results were 1 to 5 % further
    // off than those of four.
    using Sum = std::conditional_t<(W > 4), double, float>;
    Sum l = 0, acc[kA] = {};
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      const float f = __builtin_amdgcn_exp2f(red_m[w][row] - m);   // a wavefront without a visible key: 0
      const vvec x = *(const vvec*)(red_o + (size_t)(w * kRows + row) * kRedStride + d);
      l += (Sum)f * red_l[w][row];
#pragma unroll
      for (int a = 0; a < kA; ++a) acc[a] += (Sum)f * x[a];
    }
    vvec y;
#pragma unroll
    for (int a = 0; a < kA; ++a) y[a] = (float)(acc[a] / l);
    *(vvec*)((float*)p.out + (out_row + (size_t)row * p.Hq) * D + d) = y;
  }
}

// ---- long suffixes ----------------------------------------------------------------------------------
// One workgroup per 128 rows, 32 to a wavefront, D = 64.  Splitting takes 5.5 vector
// instructions per value, so the workgroup splits a block of 32 keys once and shares the pieces through LDS, in the order the matrix
// instruction reads them:
//   K: [piece][chunk of 8 d][key], 16 bytes each: lane (key l32, half) of step t reads chunk 2 t + half.
//   V: [piece][chunk of 8 keys][d], 16 bytes each; chunk 2 g + h holds keys 4 h .. + 3 and 8 + 4 h .. + 3 of 16-key group g,
//      the keys whose weights half h of a wavefront holds in its score registers 8 g .. 8 g + 7.
// Two blocks of 32 keys are under way at once: the scores of block i + 1 run on the matrix cores beside the softmax of block i and the
// splitting of its weights, the output products of block i beside the splitting of K(i + 2) and V(i + 1) and the sums of the output.  Two
// buffers of K and two of V, one barrier a block; two workgroups to a compute unit.
// What bounds it: issue, with two wavefronts on a SIMD and their waits (48 matrix instructions, 36 reads of LDS, 310 vector and 80 scalar
// instructions a block), the loads of raw rows, which are requested at the very end of a block, and the clock under that load.  64 requests x 1070
// rows x 8 heads behind 128 keys 575 us, 656 with one block at a time, splitting between two barriers and a maximum per block; 8 x 2000 rows 260 ->
// 190, 32 x 290 behind 256 85 -> 65.  The six products alone are 302 of 64 x 1070 at the rate the instruction holds on random operands; constant
// values take 0.83 of the time, without loads (wrong) it is 0.76, with requests one after the other (Item::find) 1.03, with 256 rows and eight
// wavefronts to a workgroup, one to a unit, 1.16 (a quarter of the wavefronts wait at the diagonal).
constexpr int kBigRows = kRows * kWaves;
template <bool kStep>
__device__ __forceinline__ void attn_f32_tile(const SkvAttnF32Params& p, int block_id) {
  constexpr int D = 64;
  constexpr int kT = D / 16;             // steps of the score product
  constexpr int kA = D / 32;             // output accumulators
  constexpr int kBuf = kPieces * kKeys * D / 8;              // 16-byte chunks of a block of K, or of V
  constexpr int kRedStride = D + 4;                          // floats per query row of a result in LDS
  static_assert(kBigRows * kRedStride / 4 <= 4 * kBuf);
  __shared__ u32x4 smem[4 * kBuf + kBigRows * D / 8];
  u32x4* const k_lds = smem;
  u32x4* const v_lds = smem + 2 * kBuf;
  u32x4* const q_lds = smem + 4 * kBuf;  // Q's last pieces, [wavefront][step][lane]: in registers they would be 16 too many
  float* const red_o = (float*)smem;     // the results, after the loop

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l32 = lane & 31, half = lane >> 5;

  Item it;
  if (!it.find_by_number<kBigRows, kStep>(p, block_id)) return;
  const int h = it.h, hk = it.hk, r = it.r, qbase = it.qbase, S = it.S, L = it.L, row0 = it.row0, row1 = it.row1;
  const int key_end = L + row1;                               // keys [0, key_end) are seen by some row of the tile
  const int n_blocks = (key_end + kKeys - 1) / kKeys;
  const float c = p.scale * kLog2e;
  // this wavefront's rows and keys
  const int row_w = row0 + kRows * wave;
  const int key_end_w = row_w < row1 ? L + min(row1, row_w + kRows) : 0;
  const int seen = L + row_w;

  // ---- a block's raw values: wavefronts 2 g and 2 g + 1 take 16-key group g, whose rows lie in one page or behind one another in the
  // new rows: half the chunks of each of its K rows, half its V rows
  const int group = wave >> 1, hh = wave & 1;
  const int kg = lane & 15, kc = (lane >> 4) + 4 * hh;        // K: key of the group, chunk
  // Page ids of this wavefront's group for 64 blocks, one per lane, and for the 64 after them (a load of the id on its own,
  // behind a block's loads, would be waited for together with them).
  auto window = [&](int w) __attribute__((always_inline)) {
    const int g = 2 * (64 * w + lane) + group;
    return (int64_t)g * SKV_BLOCK_TOKENS < L && g < p.max_blocks ? p.page_table[(size_t)r * p.max_blocks + g] : -1;
  };
  int win = 0, win_cur = window(0), win_nxt = window(1);      // windows win and win + 1
  // The group's rows of a block as a buffer that ends where they do: those behind, and an absent page, read as zeros.  K asks a block ahead
  // of V, which finds the place worked out.
  const unsigned row_bytes = (unsigned)p.Hkv * D * 4u;
  const uint64_t kpool_a = (uint64_t)p.kpool, vpool_a = (uint64_t)p.vpool, knew_a = (uint64_t)p.knew, vnew_a = (uint64_t)p.vnew;
  struct Rows {
    uint64_t k, v;
    int bytes;
  } k_rows;
  auto uniform = [](uint64_t x) __attribute__((always_inline)) {
    return (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(x >> 32)) << 32 | (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)x);
  };
  auto rows_of = [&](int b) __attribute__((always_inline)) {
    const int page = __builtin_amdgcn_readlane((b >> 6) == win ? win_cur : win_nxt, b & 63);
    const int key0 = b * kKeys + 16 * group;
    const bool old = key0 < L;
    const int n = old ? (page >= 0 && page < p.n_pages ? 16 : 0) : max(0, min(16, key_end - key0));
    const int64_t row = old ? (int64_t)page * SKV_BLOCK_TOKENS : qbase + key0 - L;
    const uint64_t at = n ? (uint64_t)(row * p.Hkv + hk) * (D * 4) : 0;
    return Rows{(old ? kpool_a : knew_a) + at, (old ? vpool_a : vnew_a) + at, n ? (int)((n - 1) * row_bytes) + D * 4 : 0};
  };
  auto buffer = [&](uint64_t at, int bytes) __attribute__((always_inline)) {   // (a descriptor that is not scalar costs a loop around each load)
    return __builtin_amdgcn_make_buffer_rsrc((void*)uniform(at), 0, __builtin_amdgcn_readfirstlane(bytes), 0x00020000);
  };
  const unsigned k_off = (unsigned)kg * row_bytes + kc * 32u, v_off = (unsigned)(4 * hh) * row_bytes + lane * 4u;
  float kraw[8], vraw[8];
  auto load_k = [&](int b) __attribute__((always_inline)) {
    k_rows = rows_of(b);
    const auto rsrc = buffer(k_rows.k, k_rows.bytes);
    const f32x4 x = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, k_off, 0, 0));
    const f32x4 y = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, k_off + 16, 0, 0));
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      kraw[i] = x[i];
      kraw[4 + i] = y[i];
    }
  };
  auto load_v = [&](const Rows& x) __attribute__((always_inline)) {
    const auto rsrc = buffer(x.v, x.bytes);
    unsigned at = v_off;   // (the row in the lane's offset: the range check takes a scalar one off the buffer's size, which may be less)
    asm volatile("" : "+v"(at));   // (each from the one before: eight kept through the loop would be spilled)
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      vraw[i] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rsrc, at, 0, 0));
      at += (i == 3 ? 5 : 1) * row_bytes;
    }
  };
  // (not in front of the branches around what is done with them: everybody would wait there for what has just been requested)
  auto here = [](float (&x)[8]) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < 8; ++i) asm volatile("" : "+v"(x[i]));
  };
  u32x4* const k_dst = k_lds + kc * kKeys + 16 * group + kg;
  u32x4* const v_dst = v_lds + wave * D + lane;
  const u32x4* const k_src = k_lds + half * kKeys + l32;
  const u32x4* const v_src = v_lds + half * D + l32;

  load_k(0);
  load_v(k_rows);

  // ---- Q pieces (B operand): lane (query l32, half), step t: d = 16 t + 8 half .. + 7
  bf16x8 qp[kT][2];
  u32x4* const q_last = q_lds + wave * (kT * 64) + lane;
  RangeOfQ q_range;
  {
    const float* src = (const float*)p.q + ((size_t)(qbase + min(row_w + l32, S - 1)) * p.Hq + h) * D + 8 * half;
#pragma unroll
    for (int t = 0; t < kT; ++t) {
      const f32x4 a = *(const f32x4*)(src + 16 * t), b = *(const f32x4*)(src + 16 * t + 4);
      const float x[8] = {a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]};
#pragma unroll
      for (int k = 0; k < 8; ++k) q_range.add(x[k]);
      const Pieces q = split8(x);
      qp[t][0] = q.p[0];
      qp[t][1] = q.p[1];
      q_last[t * 64] = __builtin_bit_cast(u32x4, q.p[2]);   // (read by this lane only)
    }
  }
  auto store_k = [&](int buf) __attribute__((always_inline)) {
    const Pieces k = split8(kraw);
#pragma unroll
    for (int q = 0; q < kPieces; ++q) k_dst[buf * kBuf + q * (D / 8) * kKeys] = __builtin_bit_cast(u32x4, k.p[q]);
  };
  auto store_v = [&](int buf) __attribute__((always_inline)) {
    const Pieces v = split8(vraw);
#pragma unroll
    for (int q = 0; q < kPieces; ++q) v_dst[buf * kBuf + q * (kKeys / 8) * D] = __builtin_bit_cast(u32x4, v.p[q]);
  };
  auto publish = [&]() __attribute__((always_inline)) {   // (loads from memory stay in flight)
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };

  f32x16 o[kA];   // O^T: d = 32 a + 8 (e / 4) + 4 half + e % 4, query l32
#pragma unroll
  for (int a = 0; a < kA; ++a)
#pragma unroll
    for (int e = 0; e < 16; ++e) o[a][e] = 0.f;
  float m_ref = -INFINITY, l_run = 0.f;   // reference (scaled, exp2 units) and this half's running sum, per query
  const f32x16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  struct Scores {
    f32x16 s, low;
  } sc[2];
  sc[0].s = sc[0].low = sc[1].s = sc[1].low = zero16;
  // Fragments of K, then of V: a piece's registers take the next step's as soon as it has been used (two sets spilled Q's pieces, and a
  // reload waits for every load in flight).
  bf16x8 frag[kPieces];
  auto k_piece = [&](int buf, int t, int q) __attribute__((always_inline)) { frag[q] = __builtin_bit_cast(bf16x8, k_src[buf * kBuf + (q * (D / 8) + 2 * t) * kKeys]); };
  auto v_piece = [&](int buf, int a, int g, int q) __attribute__((always_inline)) {
    frag[q] = __builtin_bit_cast(bf16x8, v_src[buf * kBuf + (q * (kKeys / 8) + 2 * g) * D + 32 * a]);
  };
  auto active = [&](int i) __attribute__((always_inline)) { return i * kKeys < key_end_w; };   // block i of 32 keys

  // Scores of a block, beside `side(j)`, j = 0 .. 23: what the vector unit does behind the j-th matrix instruction.  vbuf: whose first
  // fragments are read behind them.
  auto scores = [&](int buf, int vbuf, Scores& x, auto&& side) __attribute__((always_inline)) {
#pragma unroll
    for (int q = 2; q >= 0; --q) k_piece(buf, 0, q);
    bf16x8 q2 = __builtin_bit_cast(bf16x8, q_last[0]);
#pragma unroll
    for (int t = 0; t < kT; ++t) {
#pragma unroll
      for (int n = 0; n < 6; ++n) {
        constexpr int kk[6] = {2, 1, 1, 0, 0, 0}, qq[6] = {0, 1, 0, 2, 1, 0};   // the largest apart
        f32x16& acc = n < 5 ? x.low : x.s;
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag[kk[n]], qq[n] == 2 ? q2 : qp[t][qq[n] & 1], t == 0 && (n == 0 || n == 5) ? zero16 : acc, 0, 0, 0);
        if (n == 0 || n == 2 || n == 5) {
          if (t + 1 < kT) k_piece(buf, t + 1, kk[n]);
          else v_piece(vbuf, 0, 0, kk[n]);
        }
        if (n == 3 && t + 1 < kT) q2 = __builtin_bit_cast(bf16x8, q_last[(t + 1) * 64]);
        side(6 * t + n);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  };
  // Weights of a block in 24 pieces of vector work: exponentials against the reference as it stands (0 .. 7), the reference moved where
  // they sum to too much, the weights split (8 .. 23; a pair in two steps).
  Words w[2];   // 16-key group g of the block
  float x[16], sum[2], alpha = 1.f;   // alpha: what the output so far is to be multiplied by (here, in a branch of its own, it would be copied every time)
  auto soften = [&](int j, Scores& cur) __attribute__((always_inline)) {
    if (j == 0) {
      sum[0] = sum[1] = 0.f;
      asm volatile("" : "+v"(m_ref));   // (or what the two forms below have in common is worked out in front of them, into 16 registers more)
    }
    if (j < 8) {
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        x[2 * j + k] = weight(cur.s[2 * j + k], cur.low[2 * j + k], c, m_ref);
        sum[k] += x[2 * j + k];
      }
      return;
    }
    if (j == 8) {
      const bool trip = !(sum[0] + sum[1] <= kSumLimit);
      alpha = 1.f;
      if (__builtin_expect(__any(trip), 0)) alpha = move_reference(cur.s, cur.low, trip, c, x, sum, m_ref, l_run);
      l_run += sum[0] + sum[1];
    }
    const int pair = (j - 8) >> 1;
    split_step(x[2 * pair], x[2 * pair + 1], j & 1, pair & 3, w[pair >> 2]);
  };
  // O^T += V^T P^T of a block: summed from zero, small products first, and added once; beside late(j), j = 0 .. 23, and the sums.
  // (in place: the compiler sums into the block's registers and copies them back; nor does it see what the matrix core has not written yet)
  auto add_to = [&](f32x16& y, int e, const f32x16& add) __attribute__((always_inline)) {
    float x = y[e];
    asm volatile("v_fma_f32 %0, %0, %1, %2" : "+v"(x) : "v"(alpha), "v"(add[e]));
    y[e] = x;
  };
  auto output = [&](int buf, auto&& late) __attribute__((always_inline)) {
    f32x16 add[kA];
#pragma unroll
    for (int a = 0; a < kA; ++a) {
      bf16x8 first;   // the first group's largest piece waits for the second's small products
#pragma unroll
      for (int n = 0; n < 12; ++n) {
        constexpr int vv[12] = {2, 1, 1, 0, 0, 2, 1, 1, 0, 0, 0, 0}, ww[12] = {0, 1, 0, 2, 1, 0, 1, 0, 2, 1, 0, 0};
        const int g = n < 5 || n == 10 ? 0 : 1;
        add[a] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(n == 10 ? first : frag[vv[n]], __builtin_bit_cast(bf16x8, w[g][ww[n]]), n == 0 ? zero16 : add[a], 0, 0, 0);
        if (n == 4) first = frag[0];
        if (n == 0 || n == 2 || n == 4) v_piece(buf, a, 1, vv[n]);
        if (a + 1 < kA && (n == 5 || n == 7 || n == 11)) v_piece(buf, a + 1, 0, vv[n]);
        late(12 * a + n);
        if (a == 1 && n >= 4) {
#pragma unroll
          for (int e = 2 * (n - 4); e < 2 * (n - 4) + 2; ++e) add_to(o[0], e, add[0]);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    asm volatile("s_nop 7\n\ts_nop 7\n\ts_nop 1" : "+v"(add[1]));
#pragma unroll
    for (int e = 0; e < 16; ++e) add_to(o[1], e, add[1]);
  };
  auto nothing = [](int) __attribute__((always_inline)) {};
  auto idle = [&](Scores& z) __attribute__((always_inline)) {   // for the last score instructions, whose readers may sit behind a branch
    asm volatile("s_nop 7\n\ts_nop 7\n\ts_nop 1" : "+v"(z.s), "+v"(z.low));
  };
  // Block i, kB = i % 2.  (Behind the last one stale values are split and rows read again, for nobody.)
  auto block = [&]<int kB>(int i) __attribute__((always_inline)) {
    Scores &cur = sc[kB], &nxt = sc[kB ^ 1];
    Words kw, vw;
    const Rows v_rows = k_rows;   // of block i + 2
    auto late = [&](int j) __attribute__((always_inline)) {
      if (j == 0) here(kraw);
      if (j == 12) here(vraw);
      if (j < 8) split_step(kraw[j & ~1], kraw[j | 1], j & 1, j >> 1, kw);
      else if (j < 11) k_dst[kB * kBuf + (j - 8) * (D / 8) * kKeys] = kw[j - 8];
      else if (j >= 12 && j < 20) split_step(vraw[(j - 12) & ~1], vraw[(j - 12) | 1], j & 1, (j - 12) >> 1, vw);
      else if (j >= 20 && j < 23) v_dst[(kB ^ 1) * kBuf + (j - 20) * (kKeys / 8) * D] = vw[j - 20];
    };
    if (active(i)) {
      mask(cur.s, cur.low, i * kKeys, seen);
      if (active(i + 1)) {
        scores(kB ^ 1, kB, nxt, [&](int j) __attribute__((always_inline)) { soften(j, cur); });
      } else {
#pragma unroll
        for (int q = 2; q >= 0; --q) v_piece(kB, 0, 0, q);
#pragma unroll
        for (int j = 0; j < 24; ++j) soften(j, cur);
      }
      output(kB, late);
    } else {
#pragma unroll
      for (int j = 0; j < 24; ++j) late(j);
    }
    // (requested in either branch the values would be copied behind it, and the copies wait for them)
    load_k(i + 3);
    load_v(v_rows);
    if (((i + 3) >> 6) != win) {
      ++win;
      win_cur = win_nxt;
      win_nxt = window(win + 1);
      asm volatile("" : "+v"(win_nxt));   // (waited for here and not wherever it may be copied)
    }
    if (i + 1 < n_blocks) publish();
  };

  // ---- prologue: K(0), K(1), V(0) in LDS; scores of block 0, whose row maxima are the first reference
  store_k(0);
  load_k(1);
  store_v(0);
  load_v(k_rows);
  store_k(1);
  load_k(2);
  publish();
  if (active(0)) {
    scores(0, 0, sc[0], nothing);
    idle(sc[0]);
    mask(sc[0].s, sc[0].low, 0, seen);
    m_ref = fmaxf(over_halves(largest(sc[0].s, sc[0].low), SkvMax()) * c, -3.0e38f);   // (a row sees key 0)
  }
  publish();   // (K(2) takes the place of K(0))
  for (int i = 0; i < n_blocks; i += 2) {
    block.template operator()<0>(i);
    if (i + 1 >= n_blocks) break;
    block.template operator()<1>(i + 1);
  }
  asm volatile("s_nop 7\n\ts_nop 3");
  l_run = over_halves(l_run, SkvAdd());

  const bool no_pieces = q_range.odd() || !all_finite(o, l_run), small = some_small(o, l_run);
  if (__builtin_expect(__syncthreads_or(no_pieces || small), 0)) {
    if (__syncthreads_or(no_pieces || tiny_columns<D, kWaves>(p, it))) {
      rows_one_by_one<D, kWaves>(p, it);
      return;
    }
  }
  // ---- output, through LDS: whole rows leave together
  {
    // o / l_run: a product and, once, what it leaves, rounded as a division is (the same bits in 86 M results; the sums are a row's weights, 1 to
    // 2^31), in a third of its instructions: 64 requests of 1070 rows 594 us, divided 602, 19 of 200 behind 320 40.0 / 41.0
    const float inv = 1.f / l_run;
    auto over = [&](float x) __attribute__((always_inline)) {
      const float y = x * inv;
      return __builtin_fmaf(__builtin_fmaf(-y, l_run, x), inv, y);
    };
    float* dst = red_o + (size_t)(kRows * wave + l32) * kRedStride + 4 * half;
#pragma unroll
    for (int a = 0; a < kA; ++a)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        *(f32x4*)(dst + 32 * a + 8 * i) = f32x4{over(o[a][4 * i]), over(o[a][4 * i + 1]), over(o[a][4 * i + 2]), over(o[a][4 * i + 3])};
  }
  __syncthreads();
  float* out = (float*)p.out + (((size_t)qbase + row0) * p.Hq + h) * D;
  for (int i = threadIdx.x; i < (row1 - row0) * (D / 4); i += kThreads)
    *(f32x4*)(out + (size_t)(i / (D / 4)) * p.Hq * D + i % (D / 4) * 4) = *(const f32x4*)(red_o + (size_t)(i / (D / 4)) * kRedStride + i % (D / 4) * 4);
}

// ---- one row per request ---------------------------------------------------------------------------
// A wavefront per row and head in plain arithmetic: the tiles above are 32 rows, whatever a request has.
template <int D>
__global__ __launch_bounds__(kThreads, D == 64 ? 3 : 1) void attn_f32_rows_kernel(SkvAttnF32Params p) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t at = (int64_t)blockIdx.x * kWaves + wave;
  const int tok = (int)(at / p.Hq);
  if (tok >= min(p.max_rows, (int64_t)p.q_off[p.n_req])) return;
  int r = 0;   // the last request that starts at or before the row
  for (int n = p.n_req; n > 1;) {
    const int step = (n + 63) / 64, idx = r + lane * step;
    const int k = __builtin_popcountll(__ballot(idx < r + n && p.q_off[idx] <= tok));
    const int lo = r + (k > 0 ? k - 1 : 0) * step;
    n = min(step, r + n - lo);
    r = lo;
  }
  r = __builtin_amdgcn_readfirstlane(r);
  const int L = __builtin_amdgcn_readfirstlane(p.matched_len[r]);
  const Row row = {r, L > 0 ? L & ~(SKV_BLOCK_TOKENS - 1) : 0, __builtin_amdgcn_readfirstlane(p.q_off[r]), tok, (int)(at % p.Hq)};
  one_row<D, D>(p, row);
}

// Tiles of 128 rows (d 64; `items`: of 32 rows, `alone`: a wavefront takes one by itself).  Always where requests have two full tiles on average and
// these fill the places of the chip: 532 such calls 0.80 of the time of 32-row items, 2 slower by 2 % and more. Else 32-row items share out fewer
// rows than a tile holds, and few of them, better; and alone they have nothing to merge, which pays where keys are few.  So for items enough whose
// rows fill three quarters of their tiles, or half where the tiles are one round of the chip's 512 places (behind the first round half-filled tiles
// cost most).  us with 32 rows to an item / so: 64 requests of 64 rows behind 256 keys, 8 heads over 8, 512 tiles, 37.4 / 32.2, 8 of 140, 32 over 8,
// 35 / 27; but 55 of 64 behind up to 1500, 16 over 4, 880 tiles, 111 / 153, 66 of 87 behind 1700, 8 over 8, 528 tiles, 181 / 208 (round); 28 of 182
// behind up to 4200, 8 over 8, 200 / 247, 24 of 35, 4 of 8, behind 2300 61 / 102 (rows); 3 of 790, 16 over 4, 1232 items, 46 / 58, 4 of 287 behind
// 198, 32 over 8, 1248 items, 37 / 33 (items, by keys); 49 of 203, 8 over 8, 224 keys, 48 / 38, 67 of 187, 192 keys, 44 / 50, 290 of 150, 32 over 8,
// 176 keys, 510 / 638 (alone: keys, the more the more there are to do). 3000 calls of 2 to 200 requests of 40 to 1500 rows behind up to 6000 keys,
// other ones than these lines were drawn from: 0.935 of the time of 32-row items, 0.925 were every choice right, 8 slower by 5 % and more, 2 by 10
// (0.938, 41 and 16 with half-filled tiles in any number); lengths that differ are not known here.
bool large_tiles(const SkvAttnF32Params& p, int64_t items, bool alone) {
  const int64_t full = p.max_rows / kBigRows, rows = (p.max_rows + p.n_req - 1) / p.n_req, tiles = (rows + kBigRows - 1) / kBigRows;
  if (full >= 2 * (int64_t)p.n_req && full * p.Hq >= 512) return true;
  const int64_t keys = std::max<int64_t>(rows, (int64_t)p.max_blocks * SKV_BLOCK_TOKENS), workgroups = p.n_req * tiles * p.Hq;
  if (alone) return 100 * rows > 65 * kBigRows * tiles && keys > 160 + std::min<int64_t>(workgroups, 4096) / 20;
  const bool round = workgroups > 448 && workgroups <= 512;
  return (round ? 2 * rows >= kBigRows * tiles : 4 * rows >= 3 * kBigRows * tiles) && items >= (keys > 512 ? 1408 : 1088);
}

// What a launch carries behind its attention's workgroups: the rest of a step of up to 64 requests (a lane each).  It needs nothing of the
// attention, nor that anything of it but q_off, which the workgroups work out (Item::rows_end).  So a step has one launch less, and short
// workgroups to fill the places that the last long ones leave: eight requests of 270 rows behind 50 keys 28.0 -> 24.7 us a pass, 64 of 1080
// 583 -> 567.  Not where items are so many that a wavefront takes one: those workgroups are too small to copy pages.
struct Rest {
  SkvGather gather;
  int32_t* q_off;
  SkvCount count;
  int n_attn, n_count;
};
template <int W>
__device__ __forceinline__ void rest_of_step(const SkvAttnF32Params& p, const Rest& x, int block) {
  __shared__ int64_t first[kSkvGatherScan + 1];
  if (block == 0) {
    int own;
    const int lane = threadIdx.x, end = Item::rows_end(p, own);
    if (lane == 0) x.q_off[0] = 0;
    if (lane < p.n_req) x.q_off[lane + 1] = end;
  } else if (block <= x.n_count) {
    skv_count_request(x.count, block - 1);
  } else {
    const int others = x.n_attn + 1 + x.n_count;
    skv_gather_pages<true, true, 64 * W, 32 / W>(x.gather, (int)blockIdx.x - others, (int)gridDim.x - others, first, x.gather.kpool, x.gather.vpool,
                                                 x.gather.matched_len, x.gather.page_table, x.gather.ctx_off, x.gather.kctx, x.gather.vctx);
  }
}
template <int D, int W, bool kStep>
__global__ __launch_bounds__(64 * W, D == 64 ? 2 : 1) void attn_f32_kernel(SkvAttnF32Params p, std::conditional_t<kStep, Rest, int> x) {
  if constexpr (kStep)
    if ((int)blockIdx.x >= x.n_attn) return rest_of_step<W>(p, x, (int)blockIdx.x - x.n_attn);
  attn_f32_item<D, W, kStep>(p, blockIdx.x);
}
template <bool kStep>
__global__ __launch_bounds__(kThreads, 2) void attn_f32_tile_kernel(SkvAttnF32Params p, std::conditional_t<kStep, Rest, int> x) {
  if constexpr (kStep)
    if ((int)blockIdx.x >= x.n_attn) return rest_of_step<kWaves>(p, x, (int)blockIdx.x - x.n_attn);
  attn_f32_tile<kStep>(p, blockIdx.x);
}

}  // namespace

// Whether it does.  The copy there has the attention's registers and LDS: it gets few places while the items hold most, and behind them it has fewer
// bytes in flight than in a launch of its own.  That costs more than the launch saves where it is large and the attention is bound by memory itself,
// with few rows.  us in front / with the attention.  Eight wavefronts to an item (256 places), up to 16 rows, pages of 8 KB: 55 requests, 224 items,
// 4 MB a pool 17.2 / 14.1, 9 MB 21.5 / 24.5, 17 MB 33 / 38, 154 MB 194 / 224; 37, 156 items, 28 MB 49.0 / 52.5, and 0.85 of the time below that;
// pages of 32 KB: 16, 128 items, 242 MB 267 / 222, 24, 192 items 347 / 363, 29, 232 items 403 / 450, 27, 232 items, 15 MB 23.4 / 25.3.  More rows, 8
// KB: 13 of 121, 248 items, 33 MB 104 / 117; 32 KB 0.75 to 0.93. Four (512 places), up to 16 rows: 41, 368 items, 169 MB 201 / 163; 46, 464 items,
// 484 MB 457 / 495, 61, 504 items, 21 MB 27 / 30; more rows 0.81 to 0.95.  3435 steps: 0.809 of the time in front with and without this rule, slower
// by more than 2 % 6 and 45 of them, by more than 10 % 0 and 21.
bool rest_rides(const SkvAttnF32Params& p, const SkvGather& g, int head_dim, bool large, bool eight, int64_t items) {
  if (head_dim != 64 || large) return true;
  const int64_t page_bytes = (int64_t)g.page_vec * 16, bytes = std::min((int64_t)p.n_req * p.max_blocks, g.cap_pages) * page_bytes;
  const bool few = p.max_rows <= 16 * (int64_t)p.n_req, small = page_bytes < 16384;
  if (!eight) return !few || items <= 440 || bytes < 12 << 20;
  return items <= 160 || bytes < (small ? 6 : items <= 208 ? 48 : 12) << 20 || (!few && (!small || items <= 224));
}

// Where the items fill the chip by themselves, one wavefront takes each: four times as many at once, nothing to merge.  256 / 1000
// requests of one row, 8 heads, d 64, behind no keys 25.7 / 84.6 us with four, 12.4 / 31.6 with one; behind 96 33.4 / 132 and 28.5 /
// 95; behind 480 99.9 / 390 and 106 / 385, so up to two rounds the width of the table decides.  Single rows in such numbers are
// better off without tiles: 12.7 / 20.9, 24.5 / 85, 102 / 362 (two rows each behind 96 keys: 39.3 / 135 against 28.5 / 99).
// Where every item has a compute unit to itself eight wavefronts share its keys (d 64; at 128 a SIMD holds one): 8 requests of 72 rows
// behind 256, 8 heads, 12.5 us with four, 11.9 with eight; one of 64 behind 2048 37.0 / 31.9, 2 of 300 behind 1000 28.4 / 25.1; 16 of 64
// behind 256, 384 items, 16.1 / 20.7.  Up to 256 keys, a block of 32 for each of the eight, the four have two at most and fewer states to
// merge: one of 40 behind 80 7.0 / 7.7, 16 of 33 behind 208 9.7 / 10.3 (behind 272 11.7 either way).
int skv_attn_f32_enqueue(const SkvAttnF32Params& params, int head_dim, const SkvStepRest* rest, void* stream) {
  const hipStream_t st = (hipStream_t)stream;
  SkvAttnF32Params p = params;
  const int64_t small_items = (p.max_rows / kRows + p.n_req) * p.Hq, slots = head_dim == 64 ? 2048 : 1024;   // slots: wavefronts at once
  const bool rows = small_items >= slots && 2 * p.max_rows <= 3 * (int64_t)p.n_req;
  const bool alone = small_items >= 2 * slots || (small_items >= slots && p.max_blocks <= 16) || (small_items >= slots / 2 && p.max_blocks <= 2);
  const bool large = head_dim == 64 && large_tiles(p, small_items, alone);
  const int64_t items = large ? (p.max_rows / kBigRows + p.n_req) * p.Hq : small_items;
  if (items > 0x7fffffff) {
    const int rc = rest ? skv_gather_enqueue(*rest->gather, false, rest->req_off, rest->q_off, *rest->count, stream) : SKV_OK;
    return rc ? rc : SKV_ERANGE;
  }
  const int row_groups = (int)((p.max_rows * p.Hq + kWaves - 1) / kWaves);   // (no more than items, where they are used)
  const bool eight = head_dim == 64 && items <= 256 && (p.max_blocks > 16 || p.max_rows > 256 * (int64_t)p.n_req);
  p.req_off = nullptr;
  if (rest && p.n_req <= 64 && (large || !(rows || alone)) && rest_rides(p, *rest->gather, head_dim, large, eight, items) &&
      items + 1 + p.n_req + skv_gather_blocks(*rest->gather) <= 0x7fffffff) {
    p.req_off = rest->req_off;
    const Rest x = {*rest->gather, rest->q_off, *rest->count, (int)items, rest->count->records ? p.n_req : 0};
    const int grid = (int)items + 1 + x.n_count + skv_gather_blocks(x.gather);
    if (large)
      attn_f32_tile_kernel<true><<<grid, kThreads, 0, st>>>(p, x);
    else if (eight)
      attn_f32_kernel<64, 2 * kWaves, true><<<grid, 2 * kThreads, 0, st>>>(p, x);
    else if (head_dim == 64)
      attn_f32_kernel<64, kWaves, true><<<grid, kThreads, 0, st>>>(p, x);
    else
      attn_f32_kernel<128, kWaves, true><<<grid, kThreads, 0, st>>>(p, x);
    SKV_HIP(hipGetLastError());
    return SKV_OK;
  }
  if (rest) {
    const int rc = skv_gather_enqueue(*rest->gather, false, rest->req_off, rest->q_off, *rest->count, stream);
    if (rc) return rc;
  }
  if (large)
    attn_f32_tile_kernel<false><<<(int)items, kThreads, 0, st>>>(p, 0);
  else if (head_dim == 64 && rows)
    attn_f32_rows_kernel<64><<<row_groups, kThreads, 0, st>>>(p);
  else if (head_dim == 64 && alone)
    attn_f32_kernel<64, 1, false><<<(int)items, 64, 0, st>>>(p, 0);
  else if (eight)
    attn_f32_kernel<64, 2 * kWaves, false><<<(int)items, 2 * kThreads, 0, st>>>(p, 0);
  else if (head_dim == 64)
    attn_f32_kernel<64, kWaves, false><<<(int)items, kThreads, 0, st>>>(p, 0);
  else if (rows)
    attn_f32_rows_kernel<128><<<row_groups, kThreads, 0, st>>>(p);
  else if (alone)
    attn_f32_kernel<128, 1, false><<<(int)items, 64, 0, st>>>(p, 0);
  else
    attn_f32_kernel<128, kWaves, false><<<(int)items, kThreads, 0, st>>>(p, 0);
  SKV_HIP(hipGetLastError());
  return SKV_OK;
}
