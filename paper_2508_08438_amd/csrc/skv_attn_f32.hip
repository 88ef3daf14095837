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
#include <type_traits>

#include "skv_internal.h"

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
  template <int kTileRows>
  __device__ __forceinline__ bool find(const SkvAttnF32Params& p) {
    const int lane = threadIdx.x & 63;
    h = blockIdx.x % p.Hq;
    hk = h / (p.Hq / p.Hkv);
    const int t = blockIdx.x / p.Hq;
    r = 0;
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
    S = (int)min((int64_t)(__builtin_amdgcn_readfirstlane(p.q_off[r + 1]) - qbase), p.max_rows - qbase);
    const int n_tiles = (S + kTileRows - 1) / kTileRows;
    const int k_tile = t - (qbase / kTileRows + r);
    if (k_tile < 0 || k_tile >= n_tiles) return false;
    row0 = (n_tiles - 1 - k_tile) * kTileRows;                 // the request's heaviest tile first
    row1 = min(S, row0 + kTileRows);
    L = __builtin_amdgcn_readfirstlane(p.matched_len[r]);
    L = L > 0 ? L & ~(SKV_BLOCK_TOKENS - 1) : 0;               // whole blocks only
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
// A sum over a column of V that small has values (or zeros) below 2^-95 only, were there 2^25 keys.
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

// Scores -> exponentials in place; the output moves to the new maximum where that has grown.  `seen`: the last key the
// tile's first row sees; m_run: running maximum (scaled, exp2 units), l_run: this half's running sum, per query.
template <int kA>
__device__ __forceinline__ void softmax_step(f32x16& s, const f32x16& s_low, int key0, int seen, float c, f32x16 (&o)[kA], float& m_run, float& l_run) {
  const int lane = threadIdx.x & 63, l32 = lane & 31, half = lane >> 5;
#pragma unroll
  for (int e = 0; e < 16; ++e) s[e] += s_low[e];
  if (key0 + kKeys - 1 > seen) {
#pragma unroll
    for (int e = 0; e < 16; ++e)
      if (key0 + (e >> 2) * 8 + 4 * half + (e & 3) > seen + l32) s[e] = -INFINITY;
  }
  float mx = s[0];
#pragma unroll
  for (int e = 1; e < 16; ++e) mx = fmaxf(mx, s[e]);
  mx = over_halves(mx, SkvMax()) * c;
  const float m_new = fmaxf(m_run, mx);
  const float ref = m_new == -INFINITY ? 0.f : m_new;   // no visible key so far: every term is 0
  float sum[2] = {0.f, 0.f};
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    s[e] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[e], c, -ref));
    sum[e & 1] += s[e];
  }
  if (__any(m_new != m_run)) {
    const float alpha = __builtin_amdgcn_exp2f(m_run - ref);
    l_run *= alpha;
#pragma unroll
    for (int a = 0; a < kA; ++a)
#pragma unroll
      for (int e = 0; e < 16; ++e) o[a][e] *= alpha;
  }
  m_run = m_new;
  l_run += sum[0] + sum[1];
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
template <int D, int W>
__global__ __launch_bounds__(64 * W, D == 64 ? 2 : 1) void attn_f32_kernel(SkvAttnF32Params p) {
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
  if (!it.find<kRows>(p)) return;
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
// One workgroup per 128 rows, 32 to a wavefront, D = 64.  Splitting takes 5.5 vector instructions per value, so the workgroup
// splits a 64-key tile once and shares the pieces through LDS, in the order the matrix instruction reads them:
//   K: [piece][chunk of 8 d][key], 16 bytes each: lane (key l32, half) of step t reads chunk 2 t + half.
//   V: [piece][chunk of 8 keys][d], 16 bytes each; chunk 2 g + h holds keys 4 h .. + 3 and 8 + 4 h .. + 3 of 16-key group g,
//      the keys whose weights half h of a wavefront holds in its score registers 8 g .. 8 g + 7.
// The next tile's raw values travel in registers (32 per lane) while a tile is worked on; the second workgroup of the
// compute unit covers the two barriers per tile.
// What bounds it: the six products take 302 us of 64 requests x 1070 rows x 8 heads at the rate the instruction holds on
// random operands (1.8 PFLOP/s), and little of the rest hides behind them -- without loads 568 us, without splitting K and V
// 591, without the softmax 626, matrix products and LDS reads alone 463, all of it 660.  On the fp32 matrix instruction 859,
// with the kernel above 775.
__global__ __launch_bounds__(kThreads, 2) void attn_f32_tile_kernel(SkvAttnF32Params p) {
  constexpr int D = 64;
  constexpr int kT = D / 16;             // steps of the score product
  constexpr int kA = D / 32;             // output accumulators
  constexpr int kTileRows = kRows * kWaves;
  constexpr int kKc = D / 32;            // K chunks (8 values) per lane and tile
  constexpr int kTile = 64;              // keys per LDS tile: a 16-key group (one page, or 16 new rows) per wavefront
  constexpr int kHalfTile = kPieces * kTile * D / 8;         // 16-byte chunks of K, or of V
  constexpr int kRedStride = D + 4;                          // floats per query row of a result in LDS
  constexpr int kRed = kTileRows * kRedStride / 4;  // 16-byte chunks
  __shared__ u32x4 smem[2 * kHalfTile > kRed ? 2 * kHalfTile : kRed];
  u32x4* const k_lds = smem;
  u32x4* const v_lds = smem + kHalfTile;
  float* const red_o = (float*)smem;     // the results, after the loop

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l32 = lane & 31, half = lane >> 5;

  Item it;
  if (!it.find<kTileRows>(p)) return;
  const int h = it.h, hk = it.hk, r = it.r, qbase = it.qbase, S = it.S, L = it.L, row0 = it.row0, row1 = it.row1;
  const int key_end = L + row1;                               // keys [0, key_end) are seen by some row of the tile
  const int n_tiles = (key_end + kTile - 1) / kTile;
  const float c = p.scale * kLog2e;
  // this wavefront's rows and keys
  const int row_w = row0 + kRows * wave;
  const int key_end_w = row_w < row1 ? L + min(row1, row_w + kRows) : 0;

  // ---- a tile's raw values: wavefront w takes 16-key group w, whose rows lie in one page or behind one another in the new rows
  const size_t row_len = (size_t)p.Hkv * D;
  const int kg = lane & 15, kc = lane >> 4;   // K: key of the group, first chunk
  // Page ids of this wavefront's groups for 64 tiles, one per lane, and for the 64 after them (a load of the id on its own,
  // behind a tile's loads, would be waited for together with them).
  auto window = [&](int w) __attribute__((always_inline)) {
    const int g = 4 * (64 * w + lane) + wave;
    return (int64_t)g * SKV_BLOCK_TOKENS < L && g < p.max_blocks ? p.page_table[(size_t)r * p.max_blocks + g] : -1;
  };
  int win_cur = window(0), win_nxt = window(1);
  f32x4 kraw[2 * kKc];
  float vraw[16];
  RangeOfQ q_range;
  auto load_tile = [&](int tile) __attribute__((always_inline)) {
    if (tile > 0 && (tile & 63) == 0) {
      win_cur = win_nxt;
      win_nxt = window(tile / 64 + 1);
    }
    const int page = __builtin_amdgcn_readlane(win_cur, tile & 63);
    const int key0 = tile * kTile + 16 * wave;
    const float *kb, *vb;
    int last = 15;   // rows behind it re-read it
    if (key0 < L) {
      if (page < 0 || page >= p.n_pages) {   // an absent page reads as zeros
#pragma unroll
        for (int i = 0; i < 2 * kKc; ++i) kraw[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < 16; ++i) vraw[i] = 0.f;
        return;
      }
      const size_t off = ((size_t)page * SKV_BLOCK_TOKENS * p.Hkv + hk) * D;
      kb = (const float*)p.kpool + off;
      vb = (const float*)p.vpool + off;
    } else {
      const int first = min(key0, key_end - 1);
      const size_t off = ((size_t)(qbase + first - L) * p.Hkv + hk) * D;
      kb = (const float*)p.knew + off;
      vb = (const float*)p.vnew + off;
      last = min(15, key_end - 1 - first);
    }
    const float* src = kb + min(kg, last) * row_len + 8 * kc;
#pragma unroll
    for (int i = 0; i < kKc; ++i) {
      kraw[2 * i] = *(const f32x4*)(src + 32 * i);
      kraw[2 * i + 1] = *(const f32x4*)(src + 32 * i + 4);
    }
    if (__builtin_expect(last == 15, 1)) {
#pragma unroll
      for (int i = 0; i < 16; ++i) vraw[i] = vb[i * row_len + lane];
    } else {
#pragma unroll
      for (int i = 0; i < 16; ++i) vraw[i] = vb[min(i, last) * row_len + lane];
    }
  };
  auto store_tile = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < kKc; ++i) {
      const f32x4 a = kraw[2 * i], b = kraw[2 * i + 1];
      const float x[8] = {a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]};
      const Pieces k = split8(x);
#pragma unroll
      for (int q = 0; q < kPieces; ++q) k_lds[(q * (D / 8) + kc + 4 * i) * kTile + 16 * wave + kg] = __builtin_bit_cast(u32x4, k.p[q]);
    }
#pragma unroll
    for (int hh = 0; hh < 2; ++hh) {
      float x[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) x[i] = vraw[(i >> 2) * 8 + 4 * hh + (i & 3)];
      const Pieces w = split8(x);
#pragma unroll
      for (int q = 0; q < kPieces; ++q) v_lds[(q * (kTile / 8) + 2 * wave + hh) * D + lane] = __builtin_bit_cast(u32x4, w.p[q]);
    }
  };

  load_tile(0);

  // ---- Q pieces (B operand): lane (query l32, half), step t: d = 16 t + 8 half .. + 7
  Pieces qp[kT];
  {
    const float* src = (const float*)p.q + ((size_t)(qbase + min(row_w + l32, S - 1)) * p.Hq + h) * D + 8 * half;
#pragma unroll
    for (int t = 0; t < kT; ++t) {
      const f32x4 a = *(const f32x4*)(src + 16 * t), b = *(const f32x4*)(src + 16 * t + 4);
      const float x[8] = {a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]};
#pragma unroll
      for (int k = 0; k < 8; ++k) q_range.add(x[k]);
      qp[t] = split8(x);
    }
  }

  f32x16 o[kA];   // O^T: d = 32 a + 8 (e / 4) + 4 half + e % 4, query l32
#pragma unroll
  for (int a = 0; a < kA; ++a)
#pragma unroll
    for (int e = 0; e < 16; ++e) o[a][e] = 0.f;
  float m_run = -INFINITY, l_run = 0.f;   // running maximum (scaled, exp2 units) and this half's running sum, per query
  const f32x16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  auto block = [&](int key0, int kb) __attribute__((always_inline)) {   // kb: block of 32 keys of the tile
    f32x16 s = zero16, s_low = zero16;
    __builtin_amdgcn_s_setprio(1);   // (before the vector work of the SIMD's other wavefront: 181 -> 177 us for 64 requests of 200 .. 600 rows)
#pragma unroll
    for (int t = 0; t < kT; ++t) {
      Pieces k;
#pragma unroll
      for (int q = 0; q < kPieces; ++q) k.p[q] = __builtin_bit_cast(bf16x8, k_lds[(q * (D / 8) + 2 * t + half) * kTile + kKeys * kb + l32]);
      s_low = mfma_pieces<2>(k, qp[t], s_low);
      s_low = mfma_pieces<1>(k, qp[t], s_low);
      s = mfma_pieces<0>(k, qp[t], s);
    }
    __builtin_amdgcn_s_setprio(0);
    // idle states for the last score instructions: their readers may sit behind a branch, through which the compiler does
    // not count them
    asm volatile("s_nop 7\n\ts_nop 3" : "+v"(s), "+v"(s_low));
    softmax_step(s, s_low, key0, L + row_w, c, o, m_run, l_run);
    const Pieces w[2] = {weights(s, 0), weights(s, 1)};
#pragma unroll
    for (int a = 0; a < kA; ++a) {
      Pieces v[2];
#pragma unroll
      for (int g = 0; g < 2; ++g)
#pragma unroll
        for (int q = 0; q < kPieces; ++q)
          v[g].p[q] = __builtin_bit_cast(bf16x8, v_lds[(q * (kTile / 8) + 2 * (2 * kb + g) + half) * D + 32 * a + l32]);
      add_block(o[a], v[0], v[1], w);
    }
  };

  for (int tile = 0; tile < n_tiles; ++tile) {
    if (tile > 0) __syncthreads();   // every wavefront is done with the tile before
    store_tile();
    __syncthreads();
    if (tile + 1 < n_tiles) load_tile(tile + 1);
#pragma unroll 1
    for (int kb = 0; kb < kTile / kKeys; ++kb) {
      const int key0 = tile * kTile + kKeys * kb;
      if (key0 < key_end_w) block(key0, kb);
    }
  }
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
    float* dst = red_o + (size_t)(kRows * wave + l32) * kRedStride + 4 * half;
#pragma unroll
    for (int a = 0; a < kA; ++a)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        *(f32x4*)(dst + 32 * a + 8 * i) = f32x4{o[a][4 * i], o[a][4 * i + 1], o[a][4 * i + 2], o[a][4 * i + 3]} / l_run;
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

}  // namespace

// Large tiles where suffixes fill them (256 rows on average) and there are enough for every workgroup slot of the chip: 64
// requests x 1070 rows x 8 heads 660 us against 775, 32 x 290 rows 41 against 45; below, 8 x 290 rows 28 us against 21.
// Where the items fill the chip by themselves, one wavefront takes each: four times as many at once, nothing to merge.  256 / 1000
// requests of one row, 8 heads, d 64, behind no keys 25.7 / 84.6 us with four, 12.4 / 31.6 with one; behind 96 33.4 / 132 and 28.5 /
// 95; behind 480 99.9 / 390 and 106 / 385, so up to two rounds the width of the table decides.  Single rows in such numbers are
// better off without tiles: 12.7 / 20.9, 24.5 / 85, 102 / 362 (two rows each behind 96 keys: 39.3 / 135 against 28.5 / 99).
// Where every item has a compute unit to itself eight wavefronts share its keys (d 64; at 128 a SIMD holds one): 8 requests of 72 rows
// behind 256, 8 heads, 12.5 us with four, 11.9 with eight; one of 64 behind 2048 37.0 / 31.9, 2 of 300 behind 1000 28.4 / 25.1; 16 of 64
// behind 256, 384 items, 16.1 / 20.7.  Up to 256 keys, a block of 32 for each of the eight, the four have two at most and fewer states to
// merge: one of 40 behind 80 7.0 / 7.7, 16 of 33 behind 208 9.7 / 10.3 (behind 272 11.7 either way).
int skv_attn_f32_enqueue(const SkvAttnF32Params& p, int head_dim, void* stream) {
  const hipStream_t st = (hipStream_t)stream;
  const int64_t tiles = p.max_rows / (kRows * kWaves), slots = head_dim == 64 ? 2048 : 1024;   // slots: wavefronts at once
  const bool large = head_dim == 64 && tiles >= 2 * (int64_t)p.n_req && tiles * p.Hq >= 512;
  const int64_t items = ((large ? tiles : p.max_rows / kRows) + p.n_req) * p.Hq;
  if (items > 0x7fffffff) return SKV_ERANGE;
  const bool rows = items >= slots && 2 * p.max_rows <= 3 * (int64_t)p.n_req;
  const bool alone = items >= 2 * slots || (items >= slots && p.max_blocks <= 16) || (items >= slots / 2 && p.max_blocks <= 2);
  const int row_groups = (int)((p.max_rows * p.Hq + kWaves - 1) / kWaves);   // (no more than items, where they are used)
  if (large)
    attn_f32_tile_kernel<<<(int)items, kThreads, 0, st>>>(p);
  else if (head_dim == 64 && rows)
    attn_f32_rows_kernel<64><<<row_groups, kThreads, 0, st>>>(p);
  else if (head_dim == 64 && alone)
    attn_f32_kernel<64, 1><<<(int)items, 64, 0, st>>>(p);
  else if (head_dim == 64 && items <= 256 && (p.max_blocks > 16 || p.max_rows > 256 * (int64_t)p.n_req))
    attn_f32_kernel<64, 2 * kWaves><<<(int)items, 2 * kThreads, 0, st>>>(p);
  else if (head_dim == 64)
    attn_f32_kernel<64, kWaves><<<(int)items, kThreads, 0, st>>>(p);
  else if (rows)
    attn_f32_rows_kernel<128><<<row_groups, kThreads, 0, st>>>(p);
  else if (alone)
    attn_f32_kernel<128, 1><<<(int)items, 64, 0, st>>>(p);
  else
    attn_f32_kernel<128, kWaves><<<(int)items, kThreads, 0, st>>>(p);
  SKV_HIP(hipGetLastError());
  return SKV_OK;
}
