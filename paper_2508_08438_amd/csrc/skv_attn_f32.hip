// Causal GQA prefill attention, fp32: the same result as the bf16 path (SafeKV Section 2.1 over the reused prefix and
// the request's own new rows), with fp32 products, sums and softmax throughout.
//
// Both contractions run on the fp32 matrix instruction (v_mfma_f32_32x32x2_f32, fp32 multiply-adds in fp32
// accumulators).  They are formed transposed, S^T = K Q^T and O^T = V^T P^T, so a query is a lane column: the softmax is
// a register reduction plus one exchange between the halves of the wavefront, and the accumulator registers of S^T are
// the B operand of the second product as they stand.
#include "skv_internal.h"

namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

constexpr int kRows = 32;   // query rows per wavefront
constexpr int kSplit = 4;   // wavefronts of a workgroup: each takes every fourth block of keys
constexpr int kThreads = 64 * kSplit;
constexpr int kKeys = 32;   // keys per step of a wavefront
constexpr float kLog2e = 1.4426950408889634f;

template <int N> struct vec_of;
template <> struct vec_of<2> { typedef f32x2 type; };
template <> struct vec_of<4> { typedef f32x4 type; };

__device__ inline float other_half(float x) { return __shfl_xor(x, 32); }

// A work item is (request, 32-row tile, query head): one workgroup, whose four wavefronts take every fourth 32-key block
// and merge their partial softmax states through LDS.  Splitting the keys gives a small batch four times the wavefronts
// (eight 64..300-token requests of 8 heads: 47 us a pass instead of 51 with one wavefront per tile) and costs a large one
// nothing (64 requests x 1070 rows x 8 heads: 0.91 ms a pass either way).
//
// No LDS in the loop: per 32 keys a wavefront issues D matrix instructions of 64 cycles, against which the D / 8 + 16 loads
// that fetch the same keys from L2 straight into the operand layout are cheap (without them the loop is 9 % faster); sharing
// the keys between row tiles through L1, or giving a wavefront 64 rows, changed nothing.
//   S^T: A = K, lane (key l32, half) takes d = 8 j + 4 half .. + 3 as one 16-byte load per j; component i of it is the A
//        operand of instruction (j, i), whose two k slots are d = 8 j + i and 8 j + 4 + i.  Q, in LDS, is read the same way.
//   O^T: register e of S^T holds key 8 (e / 4) + 4 half + e % 4: as B operand its k slots are that key for half 0 and 1.
//        A = V^T: lane (l32, half) takes the D / 32 elements d = (D / 32) l32 .. of that key's row in one load; element a
//        is the A operand of accumulator a, whose row m then stands for d = (D / 32) m + a.
//
// What bounds it: the fp32 matrix instruction sustains 142 TFLOP/s on random operands (157 nominal) and shares the vector
// ALU with the softmax (124 with four multiply-adds beside each).  fp32, 8/8 heads, d 64, 64 requests x 1070 uncached rows
// (86 GFLOP): 0.87 ms = 99 TFLOP/s; with one wavefront per output row and plain vector arithmetic it took 19.4 ms.
template <int D>
__global__ __launch_bounds__(kThreads, 2) void attn_f32_kernel(SkvAttnF32Params p) {
  constexpr int kJ = D / 8;        // 16-byte pieces of a K row per lane
  constexpr int kA = D / 32;       // output accumulators
  typedef typename vec_of<kA>::type vvec;
  constexpr int kRedStride = D + kA;   // floats per query row of a partial state in LDS
  constexpr int kQStride = D + 4;
  constexpr int kRed = kSplit * kRows * kRedStride, kQ = kRows * kQStride;
  __shared__ __attribute__((aligned(16))) float smem[kRed > kQ ? kRed : kQ];
  float* const q_lds = smem;    // Q while the loop runs,
  float* const red_o = smem;    // the partial outputs after it
  __shared__ float red_m[kSplit][kRows], red_l[kSplit][kRows];

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l32 = lane & 31, half = lane >> 5;

  // ---- which work item.  Request r's tiles start at q_off[r] / 32 + r: at least ceil(S_r / 32) apart, so every tile has a
  // place and the place is found from q_off alone (64 requests per step); places no tile maps to leave at once.
  const int h = blockIdx.x % p.Hq;
  const int t = blockIdx.x / p.Hq;
  int r = 0;
  for (int n = p.n_req; n > 1;) {
    const int step = (n + 63) / 64;
    const int idx = r + lane * step;
    const bool before = idx < r + n && p.q_off[idx] / kRows + idx <= t;
    const int k = __builtin_popcountll(__ballot(before));   // lane 0 always counts (t is at or behind the first place)
    const int lo = r + (k > 0 ? k - 1 : 0) * step;
    n = min(step, r + n - lo);
    r = lo;
  }
  r = __builtin_amdgcn_readfirstlane(r);
  const int qbase = __builtin_amdgcn_readfirstlane(p.q_off[r]);
  const int S = (int)min((int64_t)(__builtin_amdgcn_readfirstlane(p.q_off[r + 1]) - qbase), p.max_rows - qbase);
  const int n_tiles = (S + kRows - 1) / kRows;
  const int k_tile = t - (qbase / kRows + r);
  if (k_tile < 0 || k_tile >= n_tiles) return;
  const int row0 = (n_tiles - 1 - k_tile) * kRows;            // the request's heaviest tile first
  int L = __builtin_amdgcn_readfirstlane(p.matched_len[r]);
  L = L > 0 ? L & ~(SKV_BLOCK_TOKENS - 1) : 0;                // whole blocks only
  const int row1 = min(S, row0 + kRows);
  const int key_end = L + row1;                               // keys [0, key_end) are seen by some row of the tile
  const int n_blocks = (key_end + kKeys - 1) / kKeys;
  const int hk = h / (p.Hq / p.Hkv);
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
  // scores -> exponentials in place; the output moves to the new maximum where that has grown
  auto softmax = [&](f32x16& s, int b) __attribute__((always_inline)) {
    // idle states for the last score instruction (16 passes): its readers may sit behind a branch, through which the
    // compiler does not count them
    asm volatile("s_nop 7\n\ts_nop 7\n\ts_nop 3" : "+v"(s));
    const int key0 = b * kKeys, seen = L + row0;   // the tile's first row sees keys up to here
    if (key0 + kKeys - 1 > seen) {
#pragma unroll
      for (int e = 0; e < 16; ++e)
        if (key0 + (e >> 2) * 8 + 4 * half + (e & 3) > seen + l32) s[e] = -INFINITY;
    }
    float mx = s[0];
#pragma unroll
    for (int e = 1; e < 16; ++e) mx = fmaxf(mx, s[e]);
    mx = fmaxf(mx, other_half(mx)) * c;
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
  };
  // Q: through LDS, read as B operands from there (its registers would cost the second wavefront of the SIMD)
  for (int i = threadIdx.x; i < kRows * (D / 4); i += kThreads) {
    const int row = i / (D / 4), ch = i % (D / 4);
    *(f32x4*)(q_lds + row * kQStride + 4 * ch) =
        *(const f32x4*)((const float*)p.q + ((size_t)(qbase + min(row0 + row, S - 1)) * p.Hq + h) * D + 4 * ch);
  }
  __syncthreads();
  const float* const q_lane = q_lds + l32 * kQStride + 4 * half;
  int b = wave;
  if (b < n_blocks) {
    uint64_t ka, va;
    bool ok;
    int page_nxt = page_of(b);
    locate(b, page_nxt, ka, va, ok);
    load_k(ka, ok);
    page_nxt = b + kSplit < n_blocks ? page_of(b + kSplit) : -1;
    // One block: its V rows travel during the scores, the next block's K rows during the softmax and the output update.
    for (; b < n_blocks; b += kSplit) {
      load_v(b, va, ok);
      __builtin_amdgcn_sched_barrier(0);
      f32x16 s;
#pragma unroll
      for (int j = 0; j < kJ; ++j) {
        const f32x4 qf = *(const f32x4*)(q_lane + 8 * j);
#pragma unroll
        for (int i = 0; i < 4; ++i)
          s = __builtin_amdgcn_mfma_f32_32x32x2f32(kf[j][i], qf[i], i + j == 0 ? zero16 : s, 0, 0, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
      if (b + kSplit < n_blocks) {
        locate(b + kSplit, page_nxt, ka, va, ok);
        load_k(ka, ok);
        if (b + 2 * kSplit < n_blocks) page_nxt = page_of(b + 2 * kSplit);
      }
      softmax(s, b);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int e = 0; e < 16; ++e)
#pragma unroll
        for (int a = 0; a < kA; ++a) o[a] = __builtin_amdgcn_mfma_f32_32x32x2f32(vf[e][a], s[e], o[a], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
    asm volatile("s_nop 7\n\ts_nop 7\n\ts_nop 3");
  }
  l_run += other_half(l_run);
  __syncthreads();   // Q is no longer needed

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
    for (int w = 0; w < kSplit; ++w) m = fmaxf(m, red_m[w][row]);
    float l = 0.f;
    vvec acc = {};
#pragma unroll
    for (int w = 0; w < kSplit; ++w) {
      const float f = __builtin_amdgcn_exp2f(red_m[w][row] - m);   // a wavefront without a visible key: 0
      l += f * red_l[w][row];
      acc += f * *(const vvec*)(red_o + (size_t)(w * kRows + row) * kRedStride + d);
    }
    *(vvec*)((float*)p.out + (out_row + (size_t)row * p.Hq) * D + d) = acc / l;
  }
}

}  // namespace

int skv_attn_f32_enqueue(const SkvAttnF32Params& p, int head_dim, void* stream) {
  const int64_t items = (p.max_rows / kRows + p.n_req) * p.Hq;
  if (items > 0x7fffffff) return SKV_ERANGE;
  if (head_dim == 64)
    attn_f32_kernel<64><<<(int)items, kThreads, 0, (hipStream_t)stream>>>(p);
  else
    attn_f32_kernel<128><<<(int)items, kThreads, 0, (hipStream_t)stream>>>(p);
  SKV_HIP(hipGetLastError());
  return SKV_OK;
}
