// Causal GQA prefill attention of the uncached suffix over reused paged prefix KV plus the
// request's own new KV.
//
// SafeKV Section 2.1: inference attends over all previous tokens; with KV caching the K/V of
// the cached prefix are reused and only the new tokens' part is computed.  Row i of the
// suffix therefore attends to the L reused positions (read from the page pool through the
// page table the match produced) and to its own positions 0..i.
//
// bf16 path: flash-style streaming over 64-key tiles with online softmax in fp32; the two
// contractions (K.Q^T and V^T.P^T) run on the matrix cores (v_mfma_f32_16x16x32_bf16), the
// softmax on the vector ALU.  A workgroup of eight wavefronts (four, two workgroups to a compute unit, where items are
// short) shares every K/V tile through LDS; each wavefront owns 32 query rows, those of up to four heads at as few positions (the query heads of one
// kv head share a workgroup, so a K/V tile is fetched once for the group).  K/V rows travel global -> LDS with
// direct-to-LDS loads (no stop in registers, no LDS store instructions), six stages of 32 keys each, or five.
// The products are formed transposed (S^T = K Q^T, O^T = V^T P^T) so that a query is a
// lane-column of the MFMA accumulator: row sums are register reductions, and the P^T
// accumulator registers are already in the B-operand layout of the second product; V^T
// fragments come from the LDS transpose load.  The inner loop is a three-stage software
// pipeline over 32-key sub-tiles: the scores of sub-tile h + 1, the softmax of sub-tile h and
// the output update with sub-tile h - 1 share a half-step, in which nothing depends on
// anything else, so MFMAs and vector instructions alternate in the instruction stream.
// fp32 path: skv_attn_f32.hip.
#include <algorithm>
#include <atomic>
#include <climits>

#include "skv_gather.h"

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));

constexpr int kD = 128;          // head dim of the bf16 kernel
constexpr int kBN = 64;          // keys per LDS tile
constexpr int kStageRows = 16;   // rows of a wave's Q / O staging tile
constexpr float kSumLimit = 4096.f;   // move the softmax reference when a lane's sum over a query's 8 keys of a sub-tile exceeds this
constexpr int kRowsPerWave = 32; // query rows per wavefront
constexpr int kWaves = 8;        // two per SIMD: one wave's softmax overlaps the other's MFMAs
constexpr int kThreads = kWaves * 64;
// LDS tile layout (K and V alike): a 64-key tile is 16 segments of 4 keys, 1 KB each.  Inside segment s the
// 16-byte piece (key q of the segment, chunk c of the 256-byte row) sits at (c / 4) * 256 + q * 64 + (c % 4 ^ turn(s)) * 16.
// One direct-to-LDS load of a wavefront fills one segment: the hardware puts what lane i fetched at byte 16 i, so
// lane i fetches chunk 4 (i / 16) + (i % 4 ^ turn(s)) of key (i / 4) % 4 -- four lanes read 64 consecutive bytes of a row.
// turn() makes the fragment reads free of bank conflicts: K (ds_read_b128, 16 lanes = one chunk of 16 keys) asks for four different
// values in four segments, V^T (ds_read_b64_tr_b16, 32 lanes = 32 bytes of 4 keys in two segments) for values that differ in bit 1 in
// neighbouring ones.  The addresses of different fragments differ by constants only (V^T's by two sets of them).
constexpr int kSeg = 512;            // bf16 elements per segment
constexpr int kHalf = 8 * kSeg;      // bf16 elements per 32 keys: a stage
constexpr int kHalfBytes = kHalf * 2;
__device__ __forceinline__ int turn(int s) { return ((s >> 1) & 1) | ((s ^ (s >> 1)) & 1) << 1; }   // 0, 2, 3, 1
constexpr float kLog2e = 1.4426950408889634f;

struct AttnParams {
  const void *q, *knew, *vnew, *kpool, *vpool;
  void* out;
  const int32_t* page_table;
  const int32_t* items;      // kItemInts ints per work item
  const int32_t* n_items;
  const int32_t* splits;     // kSplitInts ints per work item whose keys are split over several workgroups
  float* partials;           // kSlotFloats floats per part and (kv head, head group); null: nothing is ever split
  int max_blocks, n_pages, Hq, Hkv;
  int heads_per_wg;          // query heads of one kv head handled by one workgroup (1, 2, 4 or 8)
  int G, n_hg;               // query heads of a kv head; its head groups
  float scale;
  // what the work list is made of, for workgroups that find their item themselves
  const int32_t *q_off, *matched_len;
  const int32_t* req_off;    // not null: q_off is still to come, they make it from this and write it
  int32_t* q_off_out;
  int32_t* splits_out;       // = splits and n_items, written by them for the merge
  int32_t* n_items_out;
  int n_req, pos_log, max_items;
  float rows_filled;
};

// ---- work list ---------------------------------------------------------------------------------
// One workgroup.  items[] lists one 32-byte record per (request, q tile) pair -- {request, first suffix row of
// the tile, first row of the request in Q, its suffix length S, its reused length L, end row of the tile, first key tile,
// part} -- so that a workgroup of the attention kernel learns everything about its piece of work from one load.  Where it
// pays (order_above) requests with the most keys come first, and of a request always its heaviest (last) tile: what runs last is short, so the chip empties evenly,
// and the tiles of a request stay together, so they find its keys in L2.  The q tiles of a request are cut so that
// L + (first row of a tile) is a multiple of the 64-key tile (or of the q tile where that is shorter): the first tile is
// short when L is not, and every later tile ends where a key tile ends, so
// no workgroup streams a key tile for the sake of a few keys of round-up -- unless the short first tile makes the
// request one tile longer than cutting from row 0 would and the reused prefix is long (L > S / 2): a tile more costs
// a pass over about L + S / 2 keys, the round-up one more 64-key iteration in each of the S / 64 tiles.
//
// Small batches leave most of the chip idle and their time is the length of one workgroup's pass over the keys (one turn
// behind 24 k cached tokens: 80 workgroups, 0.50 ms).  Their items are split along the keys: every part is a record of its
// own (part = (slot + 1) << kPartBits | key tiles), leaves its unnormalised output, reference and row sum in the workspace,
// and attn_merge_kernel combines them.  The part length c is the smallest for which all parts run in one round, or in
// two, of one workgroup per compute unit.  Forecast: whole items take 12 us + 1.27 per key tile of the longest, 0.87 where half the
// wavefronts or more have no rows; split ones 22 us, 8 for the partial states of full workgroups, and 1.7 times the tiles' time per
// compute unit; the batch is split where that is less.  E.g. 137 rows behind 2992 cached ones, 32 query heads over 8: 72 -> 33 us; 137 of
// each of 8 requests behind 1488 stay whole (49 us).
// These are figures of an earlier kernel (1105 shapes, whole and split timed).  Now (3650 shapes, each form timed) a call from a list takes
// 10.5 us + 1.31 / 0.81 whole and 17 + 9 + 1.45 split, one whose workgroups find their items 6.7 + 1.20 / 0.76 and 12 + 7 to 11 + 1.4 to 1.6:
// nearly all too high, which nearly cancels where they are compared: the choice is 0.5 % behind the best on average, 3.7 % where a kv head
// serves eight query heads or more.  Figures of its own for each of the two changed 302 choices there, 174 for the better and 88 for
// the worse.
//
// The kernel is a chain of dependent steps on one compute unit, so every step is short: requests are ordered by a histogram
// of their lengths, scans go through registers, and the search for c tries sixteen lengths at a time, one per wavefront
// (one request of 257 rows: 10 us, 18 with one length at a time; lists without a split 3.6 us).  Order by length and
// 32-row tiles: 32 requests of 264 rows behind 16..32 k keys, 64/8 heads: 7.32 -> 6.83 ms; 16 requests of 97..994 rows
// behind up to 8 k, 32/8 heads (order only): 525 -> 512 us.
constexpr int kItemInts = 8;
constexpr int kCus = 256;             // compute units = workgroups that run at once
constexpr int kMaxSlots = 2 * kCus;   // parts of a split batch, over all kv heads and head groups
constexpr int kStartTiles = 8;
constexpr int kLogFull = 8;           // query rows of a workgroup's wavefronts (logarithm)
static_assert(1 << kLogFull == kWaves * kRowsPerWave);
// 10 ns: a key tile of a workgroup with rows for more than half its wavefronts, or for less.  (tile_time counts a tile of eight heads and up
// to 16 rows as full, which it is not; counted by Packing 4 of 2573 calls change from split to whole, all for the worse, by up to 29 %:
// the figures' error again.  eight_heads counts it as half.)
constexpr int kTileFull = 127, kTileHalf = 87;
constexpr float kWholeCost = 1200.f, kSplitCost = 2200.f, kStateCost = 800.f, kSplitTime = 1.7f;   // 10 ns; the last a factor
constexpr int kPartBits = 20;         // key tiles of a part
constexpr int kSplitInts = 8;         // {first row, end row, first row of the request in Q, first slot, parts, 0, 0, 0}
constexpr int kSlotFloats = kWaves * 64 * (64 + 2);   // per wavefront and lane: 64 of O^T, reference, row sum

// (tile heights are powers of two and handed on as their logarithms: a division is a microsecond of this kernel's chain)
struct Cut {   // how one request's suffix is cut into q tiles
  int S, L, qb, head_rows, nt;
  __device__ void tile(int j, int pos_log, int& row0, int& row1) const {   // j-th tile from the front
    if (head_rows > 0 && j == 0) {
      row0 = 0;
      row1 = head_rows;
    } else {
      row0 = head_rows + ((j - (head_rows > 0 ? 1 : 0)) << pos_log);
      row1 = min(S, row0 + (1 << pos_log));
    }
  }
};
__device__ inline Cut cut_of(int q_begin, int q_end, int matched, int pos_log) {
  Cut c;
  c.qb = q_begin;
  c.S = q_end - q_begin;
  c.L = matched > 0 ? matched & ~(SKV_BLOCK_TOKENS - 1) : 0;   // whole blocks only
  const int last = (1 << pos_log) - 1, align = min(kBN - 1, last);
  c.head_rows = min(c.S, -c.L & align);                        // rows of the short first tile (0: none)
  c.nt = c.S > 0 ? (c.head_rows > 0 ? 1 : 0) + ((c.S - c.head_rows + last) >> pos_log) : 0;
  const int nt_plain = (c.S + last) >> pos_log;
  if (nt_plain < c.nt && 2 * c.L > c.S) {   // the short first tile would cost a whole extra tile: cut from row 0 instead
    c.head_rows = 0;
    c.nt = nt_plain;
  }
  return c;
}
// Parts an item of n key tiles is split into at part length c: every part but the first starts at a key that all of the
// item's rows see (key tile `last` or before), so that each part has a finite row maximum from its first keys on.
__device__ inline int parts_of(int n, int last, int c) {
  int parts = (int)((unsigned)(n + c - 1) / (unsigned)c);
  while (parts > 1 && (parts - 1) * (int)((unsigned)(n + parts - 1) / (unsigned)parts) > last) --parts;
  return parts;
}

__host__ __device__ inline int tile_time(int rows, int pos_log) {   // of a workgroup with that many rows of its q tile
  const int active = ((rows + kRowsPerWave - 1) / kRowsPerWave) << (kLogFull - pos_log);
  return active * 2 <= kWaves ? kTileHalf : kTileFull;
}
// The two forecasts.  workgroups: of the whole items; longest: the longest one's time; share: the time of all per compute unit;
// fill: query rows per row of the items' wavefronts.
__host__ __device__ inline float whole_time(float workgroups, float longest, float share) {
  const float two = share + longest / 2;
  return kWholeCost + (workgroups <= kCus || two < longest ? longest : two);
}
__host__ __device__ inline float split_time(float share, float fill) {
  return kSplitCost + kStateCost * (fill < 1.f ? fill : 1.f) + kSplitTime * share;
}

constexpr int kSchedThreads = 1024, kSchedWaves = kSchedThreads / 64;
constexpr int kBuckets = 128;

template <typename T>
__device__ inline T wave_max(T v) { return skv_over_wave(v, SkvMax()); }
template <typename T>
__device__ inline T wave_sum(T v) { return skv_over_wave(v, SkvAdd()); }
// first place whose scan value exceeds x (scan[n - 1] does)
__device__ inline int place_of(const int* scan, int n, int x) {
  int lo = 0, hi = n - 1;
  while (lo < hi) {
    const int mid = (lo + hi) >> 1;
    if (scan[mid] > x) hi = mid; else lo = mid + 1;
  }
  return lo;
}

__global__ __launch_bounds__(kSchedThreads) void attn_schedule_kernel(
    int n_req, const int32_t* __restrict__ q_off, const int32_t* __restrict__ matched_len, int pos_log, int max_items,
    int units /* workgroups per item */, int order_above /* requests are ordered by length if one is longer */,
    float rows_filled /* query rows, over the heads of a workgroup */,
    int32_t* __restrict__ n_items /* [0] items, [1] split items */, int32_t* __restrict__ items, int32_t* __restrict__ splits /* null: never split */) {
  __shared__ int scan[kSchedThreads], red[kSchedWaves], bucket[kBuckets];
  __shared__ int4 req_at[kSchedThreads];   // request, first row, rows, reused length
  __shared__ int4 item_a[kCus], item_b[kCus];   // the first records, for the split
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int listed = 0;
  for (int base = 0; base < n_req; base += kSchedThreads) {
    const int r = base + tid, n_here = min(kSchedThreads, n_req - base);
    Cut mine = {};
    if (r < n_req) mine = cut_of(q_off[r], q_off[r + 1], matched_len[r], pos_log);
    const int keys = mine.nt > 0 ? mine.L + mine.S : 0;
    // place in the order of falling length, to 1 / kBuckets of the longest
    int place = tid, longest = 0;
    if (n_here > 1 && order_above < INT_MAX) {
      const int m = wave_max(keys);
      if (lane == 0) red[wave] = m;
      if (tid < kBuckets) bucket[tid] = 0;
      __syncthreads();
      longest = wave_max(lane < kSchedWaves ? red[lane] : 0);
    }
    if (longest > order_above) {
      int b = 0, rank = 0;
      if (r < n_req) {
        b = kBuckets - 1 - (int)((float)keys * ((kBuckets - 0.5f) / (float)max(longest, 1)));
        b = max(0, min(kBuckets - 1, b));
        rank = atomicAdd(&bucket[b], 1);
      }
      __syncthreads();
      if (wave == 0) {   // exclusive scan, two buckets per lane
        const int c0 = bucket[2 * lane], c1 = bucket[2 * lane + 1];
        const int x = skv_wave_scan(c0 + c1);
        bucket[2 * lane] = x - c0 - c1;
        bucket[2 * lane + 1] = x - c1;
      }
      __syncthreads();
      place = bucket[b] + rank;
    }
    if (r < n_req) {
      scan[place] = mine.nt;
      req_at[place] = make_int4(r, mine.qb, mine.S, mine.L);
    }
    __syncthreads();
    int total;
    const int upto = skv_block_scan<kSchedThreads>(tid < n_here ? scan[tid] : 0, red, total);
    scan[tid] = upto;
    __syncthreads();
    // the chunk's items, one per thread and turn: the request is found in the scan
    for (int it = tid; it < total && listed + it < max_items; it += kSchedThreads) {
      const int at = place_of(scan, n_here, it);
      const int4 q = req_at[at];
      const Cut c = cut_of(q.y, q.y + q.z, q.w, pos_log);
      int row0, row1;
      c.tile(scan[at] - 1 - it, pos_log, row0, row1);   // the request's last tile first
      const int4 a = make_int4(q.x, row0, c.qb, c.S), b = make_int4(c.L, row1, 0, 0);
      int4* rec = (int4*)(items + (size_t)kItemInts * (listed + it));
      rec[0] = a;
      rec[1] = b;
      if (listed + it < kCus) {
        item_a[listed + it] = a;
        item_b[listed + it] = b;
      }
    }
    listed += total;
    __syncthreads();
  }
  const int n = min(listed, max_items);
  int n_out = n, n_split = 0;
  if (splits && n > 0 && n <= kCus && n * units <= kMaxSlots) {   // few items: split their keys?
    // every wavefront holds all items, four per lane
    int n_kt[kCus / 64], last[kCus / 64], longest = 0, sum = 0;
    float longest_time = 0.f, sum_time = 0.f;
#pragma unroll
    for (int k = 0; k < kCus / 64; ++k) {
      const int i = lane + 64 * k;
      n_kt[k] = last[k] = 0;
      if (i < n) {
        const int4 a = item_a[i], b = item_b[i];
        n_kt[k] = (b.x + b.y + kBN - 1) / kBN;
        last[k] = (b.x + a.y) / kBN;
        const float time = (float)n_kt[k] * tile_time(b.y - a.y, pos_log);
        longest_time = fmaxf(longest_time, time);
        sum_time += time;
      }
      longest = max(longest, n_kt[k]);
      sum += n_kt[k];
    }
    longest = wave_max(longest);
    sum = wave_sum(sum);
    longest_time = wave_max(longest_time);
    const float share = wave_sum(sum_time) * units / kCus;
    const bool worth = split_time(share, rows_filled / (n << kLogFull)) < whole_time(n * units, longest_time, share);
    if (worth) {
      // smallest part length for which all parts have room in one round (wavefronts 0 .. 7) or two (8 .. 15): eight lengths
      // between the last that did not fit and the first that did, until they meet
      const int room1 = kCus / units, room2 = 2 * kCus / units, half = wave >> 3;
      const int room = half ? room2 : room1;
      int lo1 = 1, hi1 = longest, lo2 = 1, hi2 = longest;
      if (room1 >= n) lo1 = max(1, min(longest, (sum + room1 - 1) / room1)); else lo1 = longest;
      if (room2 >= n) lo2 = max(1, min(longest, (sum + room2 - 1) / room2)); else lo2 = longest;
      int turn = 0;
      __shared__ int fits[2][kSchedWaves];
      while (lo1 < hi1 || lo2 < hi2) {
        const int lo = half ? lo2 : lo1, hi = half ? hi2 : hi1;
        const int c = lo + (int)(((long long)(hi - lo) * (wave & 7)) >> 3);   // wavefront 0 of the eight tries lo itself
        int p = 0;
  #pragma unroll
        for (int k = 0; k < kCus / 64; ++k)
          if (lane + 64 * k < n) p += parts_of(n_kt[k], last[k], c);
        p = wave_sum(p);
        if (lane == 0) fits[turn & 1][wave] = p <= room;
        __syncthreads();
        const uint64_t ok = __ballot(lane < kSchedWaves && fits[turn & 1][lane & (kSchedWaves - 1)]);
        auto narrow = [&](unsigned f, int& l, int& h) {   // f: bit k set where the k-th length fits
          if (l >= h) return;
          const int l0 = l, d = h - l, k = f ? __builtin_ctz(f) : 8;
          if (k < 8) h = l0 + (int)(((long long)d * k) >> 3);
          if (k > 0) l = l0 + (int)(((long long)d * (k - 1)) >> 3) + 1;
        };
        narrow((unsigned)ok & 255u, lo1, hi1);
        narrow((unsigned)(ok >> 8) & 255u, lo2, hi2);
        ++turn;
      }
      // one round of workgroups, which cost about kStartTiles tiles before and after their loop, or two
      const int best_c = room1 >= n && kStartTiles + hi1 <= 2 * (kStartTiles + hi2) ? hi1 : hi2;
      // scans of the parts (place in the list) and, packed, of the parts of split items (slot) and of the split items
      int4 a = {0, 0, 0, 0}, b = {0, 0, 0, 0};
      int parts = 0;
      if (tid < n) {
        a = item_a[tid];
        b = item_b[tid];
        parts = parts_of((b.x + b.y + kBN - 1) / kBN, (b.x + a.y) / kBN, best_c);
      }
      int total;
      const int mine = parts | (parts > 1 ? parts << 10 | 1 << 20 : 0);
      const int upto = skv_block_scan<kSchedThreads>(mine, red, total);
      const int n_parts = total & 1023;
      if (n_parts > n && n_parts <= max_items) {
        scan[tid] = upto & 1023;
        const int before = upto - mine, slot = (before >> 10) & 1023;
        if (parts > 1) {
          int4* sp = (int4*)(splits + kSplitInts * (before >> 20));
          sp[0] = make_int4(a.y, b.y, a.z, slot);
          sp[1] = make_int4(parts, 0, 0, 0);
        }
        if (tid < n) item_b[tid] = make_int4(b.x, b.y, parts, slot);
        __syncthreads();
        for (int it = tid; it < n_parts; it += kSchedThreads) {
          const int at = place_of(scan, n, it);
          const int4 ia = item_a[at], ib = item_b[at];
          const int j = it - (at ? scan[at - 1] : 0), kt = (ib.x + ib.y + kBN - 1) / kBN, len = (kt + ib.z - 1) / ib.z;
          int4* rec = (int4*)(items + (size_t)kItemInts * it);
          rec[0] = ia;
          rec[1] = make_int4(ib.x, ib.y, j * len, ib.z > 1 ? (ib.w + j + 1) << kPartBits | min(len, kt - j * len) : 0);
        }
        n_out = n_parts;
        n_split = total >> 20;
      }
    }
  }
  if (tid == 0) {
    n_items[0] = n_out;
    n_items[1] = n_split;
  }
}

// ---- the same list without a kernel in front of the attention -------------------------------------
// Of up to 64 requests every wavefront works its item out for itself, a request per lane and nothing through LDS: the same cuts,
// forecasts and part lengths as above (an order by length has nothing to give in one round of workgroups).  A list costs a launch and a chain of barriers, 5 to 9 us
// of every call; this 0.5 to 1.5 us of a workgroup's start, 2 to 3 where a split is searched for.  Parts fill one round of workgroups
// here: the workgroups that a second one needs room for cost every call 3 to 8 us where the parts leave it empty.
constexpr int kPlanRequests = 64, kPlanItems = 64;   // kPlanItems: a lane each, where they may be split
struct Work {
  int r, row0, row1, qbase, S, L, kt0, part;   // kt0: first key tile of the part, part: as in a record
};
// unit: kv head and head group of the caller; one of them writes what the merge reads.  False: no such item.
template <bool kParts>
__device__ __forceinline__ bool plan_item(const AttnParams& p, int item, int unit, int units, Work& w) {
  const int lane = threadIdx.x & 63;
  const bool writes = kParts && unit == 0 && threadIdx.x == 0;
  auto at_lane = [](int x, int from) __attribute__((always_inline)) { return __builtin_amdgcn_readlane(x, from); };
  auto scan = [&](int x) __attribute__((always_inline)) { return skv_wave_scan(x); };   // inclusive
  int qb = 0, qe = 0, L = 0;
  if (p.req_off) {
    if (lane < p.n_req) {
      L = p.matched_len[lane];
      qe = max(0, p.req_off[lane + 1] - p.req_off[lane] - L);
    }
    const int own = qe;
    qe = scan(own);
    qb = qe - own;
    if (item == 0 && unit == 0 && threadIdx.x < 64) {
      if (lane == 0) p.q_off_out[0] = 0;
      if (lane < p.n_req) p.q_off_out[lane + 1] = qe;
    }
  } else if (lane < p.n_req) {
    qb = p.q_off[lane];
    qe = p.q_off[lane + 1];
    L = p.matched_len[lane];
  }
  const Cut c = cut_of(qb, qe, L, p.pos_log);
  const int upto = scan(c.nt), total = at_lane(upto, 63);
  auto tile_of = [&](int own, const Cut& cut, int up) __attribute__((always_inline)) {   // the request's last tile first
    int row0, row1;
    cut.tile(up - 1 - own, p.pos_log, row0, row1);
    return int2{row0, row1};
  };
  w.kt0 = w.part = 0;
  if (!kParts || total > kPlanItems || total * units > kCus || total == 0) {   // whole items
    if (writes && item == 0) p.n_items_out[1] = 0;
    if (item >= total) return false;
    const int at = __builtin_popcountll(__ballot(upto <= item));
    const Cut mine = {at_lane(c.S, at), at_lane(c.L, at), at_lane(c.qb, at), at_lane(c.head_rows, at), at_lane(c.nt, at)};
    const int2 rows = tile_of(item, mine, at_lane(upto, at));
    w.r = at;
    w.row0 = rows.x;
    w.row1 = rows.y;
    w.qbase = mine.qb;
    w.S = mine.S;
    w.L = mine.L;
    return true;
  }
  // lane i: item i
  const int n = total;
  int at = 0, up = at_lane(upto, 0);
  Cut mine = {at_lane(c.S, 0), at_lane(c.L, 0), at_lane(c.qb, 0), at_lane(c.head_rows, 0), at_lane(c.nt, 0)};
  if (p.n_req > 1) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1)
      if (__shfl(upto, at + o - 1) <= lane) at += o;
    at = min(at, 63);
    mine = {__shfl(c.S, at), __shfl(c.L, at), __shfl(c.qb, at), __shfl(c.head_rows, at), __shfl(c.nt, at)};
    up = __shfl(upto, at);
  }
  const int2 rows = tile_of(min(lane, n - 1), mine, up);
  const bool have = lane < n;
  const int n_kt = have ? (mine.L + rows.y + kBN - 1) / kBN : 0, last = have ? (mine.L + rows.x) / kBN : 0;
  const float time = (float)n_kt * tile_time(rows.y - rows.x, p.pos_log);
  const int longest = wave_max(n_kt), sum = wave_sum(n_kt);
  const float longest_time = wave_max(have ? time : 0.f), share = wave_sum(have ? time : 0.f) * units / kCus;
  int parts = have ? 1 : 0;
  if (split_time(share, p.rows_filled / (n << kLogFull)) < whole_time(n * units, longest_time, share)) {
    // smallest part length for which all parts run in one round: sixteen lengths at a time between the last that did not fit and
    // the first that did, the items of a length dealt to four lanes
    const int room = kCus / units;
    int lo = max(1, min(longest, (sum + room - 1) / room)), hi = longest;
    while (lo < hi) {
      const int d = hi - lo, len = lo + (int)(((long long)d * (lane >> 2)) >> 4);   // the first tries lo itself
      int total_parts = 0;
      for (int i0 = 0; i0 < n; i0 += 4) {
        const int i = i0 + (lane & 3), kt = __shfl(n_kt, i & 63), la = __shfl(last, i & 63);
        if (i < n) total_parts += parts_of(kt, la, len);
      }
      total_parts += skv_dpp<kSkvQuadXor1>(0, total_parts);
      total_parts += skv_dpp<kSkvQuadXor2>(0, total_parts);
      const uint64_t fits = __ballot(total_parts <= room);
      const int k = fits ? __builtin_ctzll(fits) >> 2 : 16, l0 = lo;
      if (k < 16) hi = l0 + (int)(((long long)d * k) >> 4);
      if (k > 0) lo = l0 + (int)(((long long)d * (k - 1)) >> 4) + 1;
    }
    if (have) parts = parts_of(n_kt, last, hi);
  }
  const int part_upto = scan(parts), n_parts = at_lane(part_upto, 63);
  const bool split = n_parts > n && n_parts <= p.max_items;
  if (!split) parts = have ? 1 : 0;
  const uint64_t cut_items = __ballot(parts > 1);
  if (writes && item == 0) p.n_items_out[1] = __builtin_popcountll(cut_items);
  if (item >= (split ? n_parts : n)) return false;
  const int own = split ? __builtin_popcountll(__ballot(part_upto <= item)) : item;
  w.r = at_lane(at, own);
  w.row0 = at_lane(rows.x, own);
  w.row1 = at_lane(rows.y, own);
  w.qbase = at_lane(mine.qb, own);
  w.S = at_lane(mine.S, own);
  w.L = at_lane(mine.L, own);
  if (split) {
    const int slot_upto = scan(parts > 1 ? parts : 0);
    const int of = at_lane(parts, own), j = item - (at_lane(part_upto, own) - of), kt = at_lane(n_kt, own);
    const int len = (int)((unsigned)(kt + of - 1) / (unsigned)of), slot = at_lane(slot_upto, own) - of;
    w.kt0 = j * len;
    if (of > 1) {
      w.part = (slot + j + 1) << kPartBits | min(len, kt - j * len);
      if (writes && j == 0) {
        int4* sp = (int4*)(p.splits_out + kSplitInts * __builtin_popcountll(cut_items & ((1ull << own) - 1)));
        sp[0] = make_int4(w.row0, w.row1, w.qbase, slot);
        sp[1] = make_int4(of, 0, 0, 0);
      }
    }
  }
  return true;
}

// ---- bf16 MFMA kernel --------------------------------------------------------------------------
// max / sum of a value over the four lanes 16 apart
__device__ inline float sum_quads(float x) { return skv_over_rows(x, SkvAdd()); }
__device__ inline float max_quads(float x) { return skv_over_rows(x, SkvMax()); }

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

// A wavefront's 32 query rows: up to four heads of as few positions (lane l: head l % heads of position l / heads), so that the
// last tile of a request occupies no more wavefronts than its rows fill, and the rows of a position come and go as one
// piece of memory.
struct Packing {
  int heads_log, groups_log;   // logarithms: heads of a wavefront; wavefronts per position
  __device__ __forceinline__ void wave(int w, int row0, int& head, int& row) const {   // first head (within the workgroup's) and row
    head = (w & ((1 << groups_log) - 1)) << heads_log;
    row = row0 + ((w >> groups_log) << (5 - heads_log));
  }
};
__host__ __device__ __forceinline__ Packing packing(int heads_per_wg) {
  return heads_per_wg == 8 ? Packing{2, 1} : heads_per_wg == 4 ? Packing{2, 0} : heads_per_wg == 2 ? Packing{1, 0} : Packing{0, 0};
}

// Workgroup b runs on XCD b % 8: all work of one kv head stays on one XCD where the heads allow it, so its K/V tiles are
// re-read from that XCD's L2, and the merge finds the parts there.
__device__ __forceinline__ void unit_of_block(int b, int Hkv, int n_hg, int& item, int& kvh, int& hg) {
  // (powers of two, as a rule: three divisions one after the other are 0.4 us of a workgroup's start)
  if (((Hkv & (Hkv - 1)) | (n_hg & (n_hg - 1))) == 0) {
    const int low = min(Hkv, 8) - 1, log = __builtin_ctz(Hkv), hg_log = __builtin_ctz(n_hg);
    kvh = Hkv > 8 ? (b & 7) | ((b >> 3) & ((Hkv >> 3) - 1)) << 3 : b & low;
    const int rest = b >> log;
    hg = rest & (n_hg - 1);
    item = rest >> hg_log;
    return;
  }
  int rest;
  if (Hkv % 8 == 0) {
    const int per = Hkv / 8;
    const int xcd = b & 7, slot = b >> 3;
    kvh = xcd + 8 * (slot % per);
    rest = slot / per;
  } else {
    kvh = b % Hkv;
    rest = b / Hkv;
  }
  hg = rest % n_hg;
  item = rest / n_hg;
}

// A workgroup has the compute unit to itself or (kTwo) is one of two.
template <bool kTwo>
struct Form {
  static constexpr int waves = kTwo ? 4 : kWaves, threads = waves * 64;
  // Stages of K, and of V.  In iteration kt K's 32-key halves 2 kt + 1 .. 2 kt + 3 are in use and 2 kt + 4, 2 kt + 5 arriving, V's
  // 2 kt - 1 .. 2 kt + 1 and 2 kt + 2, 2 kt + 3: five, or six where there is room, which repeat after three tiles.
  static constexpr int halves = kTwo ? 5 : 6;
  static constexpr int loads = 16 / waves;                  // segments of a tile that a wavefront moves
  static constexpr int stage_at = kTwo ? (halves + 2) * kHalf : 2 * halves * kHalf;   // Q and O: in V's idle stages, or behind
  static constexpr int lds = kTwo ? 2 * halves * kHalf : stage_at + waves * kStageRows * kD;
};
// (not in the kernel's own text: in a template, where its arguments depend on the parameters, the host pass drops the kernel for it)
__device__ __forceinline__ void lds_load_b128(__amdgpu_buffer_rsrc_t rsrc, __bf16* dst, unsigned off) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (__attribute__((address_space(3))) void*)dst, 16, off, 0, 0, 0);
}

// kParts: the list may hold parts of items.  Without, 0.3 us less of a workgroup's start goes into what a part needs.
// kPlan: no list, the workgroup finds its item itself.
template <bool kParts, bool kPlan, bool kTwo>
__global__ __launch_bounds__(Form<kTwo>::threads, 2) void attn_bf16_kernel(AttnParams p) {
  using F = Form<kTwo>;
  constexpr int kHalves = F::halves;
  static_assert(!kTwo || !kParts);
  __shared__ __attribute__((aligned(16))) __bf16 smem[F::lds];
  __bf16* const Ks = smem;
  __bf16* const Vs = smem + kHalves * kHalf;
  // [wavefronts][16 rows][16 chunks of 8 bf16]: each wave's own staging tile for its Q rows on the way in and its O rows
  // on the way out (16 rows at a time), 16-byte chunks XOR-swizzled by row so that row-wise and fragment-wise
  // accesses are conflict free: `stage` below

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform by construction
  const int l16 = lane & 15;
  const int quad = lane >> 4;
  __bf16* stage = smem + F::stage_at + wave * (kStageRows * kD);

  // ---- which piece of work: XCD-aware decode (workgroup b runs on XCD b % 8) ----
  const int G = p.G, n_hg = p.n_hg;
  int item, kvh, hg;
  unit_of_block(blockIdx.x, p.Hkv, n_hg, item, kvh, hg);
  Work w;
  if constexpr (kPlan) {
    if (!plan_item<kParts>(p, item, kvh * n_hg + hg, p.Hkv * n_hg, w)) return;
  } else {
    // the record is read together with the item count (the grid bound keeps the index inside the list)
    const int4 rec0 = ((const int4*)(p.items + (size_t)kItemInts * item))[0];
    const int4 rec1 = ((const int4*)(p.items + (size_t)kItemInts * item))[1];
    if (item >= *p.n_items) return;
    w = {rec0.x, rec0.y, rec1.y, rec0.z, rec0.w, rec1.x, rec1.z, rec1.w};
  }
  const int kt0 = kParts ? __builtin_amdgcn_readfirstlane(w.kt0) : 0;    // first key tile of this part
  const int part = kParts ? __builtin_amdgcn_readfirstlane(w.part) : 0;  // 0: the whole item
  // Everything below counts keys from the part's first one: the reused length and with it every position shifts.
  const int L = __builtin_amdgcn_readfirstlane(w.L) - kt0 * kBN;                            // may be negative
  const int row1 = __builtin_amdgcn_readfirstlane(w.row1);                                  // end row of the q tile
  const int r = __builtin_amdgcn_readfirstlane(w.r);
  const int row0 = __builtin_amdgcn_readfirstlane(w.row0);                                  // first row of the q tile
  const int qbase = __builtin_amdgcn_readfirstlane(w.qbase);
  const int S = __builtin_amdgcn_readfirstlane(w.S);
  const int Ltot = L + S;

  const Packing pk_of = packing(p.heads_per_wg);
  const int hl_log = pk_of.heads_log;
  int head0, pos0;                                                            // first head and row of this wave
  pk_of.wave(wave, row0, head0, pos0);
  head0 += kvh * G + hg * p.heads_per_wg;
  const int n_tiles = part ? part & ((1 << kPartBits) - 1) : (L + row1 + kBN - 1) / kBN;   // 64-key tiles the workgroup streams
  const int wave_key_end = pos0 < row1 ? min(L + min(row1, pos0 + (kRowsPerWave >> hl_log)), n_tiles * kBN) : 0;  // this wave needs keys [0, wave_key_end)
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
  // (the four base addresses as values: selecting between the fields of the argument block itself makes the
  // compiler select their addresses and load through them, a vector-memory read that everything behind it waits for)
  const uint64_t kpool_a = (uint64_t)p.kpool, vpool_a = (uint64_t)p.vpool, knew_a = (uint64_t)p.knew,
                 vnew_a = (uint64_t)p.vnew;
  auto window_bases = [&](int w, int page, uint64_t& ak, uint64_t& av) __attribute__((always_inline)) {
    const int gi = w * 64 + lane;
    const int key0 = gi * SKV_BLOCK_TOKENS;
    uint64_t k = 0, v = 0;
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

  // ---- Q fragments (B operand of S^T = K Q^T): lane holds query 16 g + l16, d = 32 ks + 8 quad .. +7
  // Rows are fetched whole (16 lanes x 16 B per row) and picked up from the wave's staging tile.  The scores leave the
  // matrix core unscaled; scale * log2(e) is applied in fp32 by the multiply-add that also subtracts the reference
  // (scaling Q itself would round it to bf16 a second time: visible when scores spread over hundreds of units).
  const float c = p.scale * kLog2e;
  bf16x8 qf[2][4];   // [g][ks]
  u32x4 qv[8];
  {
    const int c16 = lane & 15;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int rr = (lane >> 4) + 4 * i;
      const int row = min(pos0 + (rr >> hl_log), S - 1);   // rows past the tile or the request are computed and dropped
      const int head = head0 + (rr & ((1 << hl_log) - 1));
      qv[i] = __builtin_nontemporal_load((const u32x4*)((const __bf16*)p.q + ((size_t)(qbase + row) * p.Hq + head) * kD + c16 * 8));
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
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) qf[pass][ks] = *(const bf16x8*)(stage + l16 * kD + (((4 * ks + quad) ^ l16) << 3));
    }
  };

  const f32x4 zero4 = {0.f, 0.f, 0.f, 0.f};
  f32x4 o[8][2];   // O^T accumulators: o[a][g][i]: d = 16 a + 4 quad + i, query 16 g + l16
#pragma unroll
  for (int a = 0; a < 8; ++a) o[a][0] = o[a][1] = zero4;

  // ---- global -> LDS, without a stop in registers ----
  // A tile is four 16-key groups; a group is one page of the pool or 16 consecutive new rows.  Each of eight wavefronts
  // moves two segments of a tile, half a group (2w and 2w + 1: keys 8w ..), each of four a group, with direct-to-LDS loads: lane i
  // fetches its piece of the segment (turn()) and the hardware puts it at slot i.  All take the
  // group's base as the buffer's and constant offsets: no vector address is formed.
  const unsigned row_bytes = (unsigned)p.Hkv * kD * 2u;
  const int seg0 = F::loads * wave;                          // this wave's first segment
  unsigned t_off[F::loads];                                  // (a scalar offset would have to lie inside the buffer)
#pragma unroll
  for (int k = 0; k < F::loads; ++k) {
    const int t_row = ((seg0 + k) & 3) * 4 + ((lane >> 2) & 3);   // row of the 16-key group this lane fetches
    t_off[k] = (unsigned)t_row * row_bytes + (unsigned)(quad * 4 + ((lane & 3) ^ turn(seg0 + k))) * 16u;
    asm volatile("" : "+v"(t_off[k]));   // (not worked out anew from its parts, which take more registers)
  }
  // Group base addresses, one 16-key group per lane for 64 groups (16 tiles, a "window"): a pool page, 16 new rows,
  // or 0 when the group has no data (past the end of the sequence, or a page id outside the pool): an empty buffer, whose rows
  // arrive as zeros.
  // A tile's bases are read with lane broadcasts.  Two consecutive windows are held; K tiles run one tile ahead of
  // V tiles, so for one iteration in sixteen K reads the later window while V still reads the earlier one.
  auto lane_bcast = [&](uint64_t x, int idx) __attribute__((always_inline)) {
    const uint32_t lo = __builtin_amdgcn_readlane((int)(uint32_t)x, idx);
    const uint32_t hi = __builtin_amdgcn_readlane((int)(uint32_t)(x >> 32), idx);
    return ((uint64_t)hi << 32) | lo;
  };
  uint64_t ak_cur, av_cur, ak_nxt, av_nxt;
  int win = 0;                       // window held in *_cur; *_nxt holds window win + 1
  window_bases(0, page_w0, ak_cur, av_cur);
  window_bases(1, page_w1, ak_nxt, av_nxt);
  const int group = seg0 >> 2;                               // 16-key group of this wave's segments
  // where they go; h: stage of the tile's first half, h_next: of its second one
  auto dst_in = [&](__bf16* stages, int h, int h_next) __attribute__((always_inline)) {
    if (!kTwo) return stages + h * kHalf + seg0 * kSeg;   // (behind one another)
    return stages + (seg0 >= 8 ? h_next : h) * kHalf + (seg0 & 7) * kSeg;
  };
  // one pool (K or V) of tile t; `base`: of the wave's group.  Where the sequence ends inside the tile so does
  // the buffer: what lies behind arrives as zeros, and the causal mask keeps it out.
  auto issue_tile = [&]<bool kWhole>(uint64_t base, int t, __bf16* dst) __attribute__((always_inline)) {
    // (the compiler clamps in vector registers, and a descriptor that is not scalar costs a loop around each load)
    const int rows = kWhole ? 16 : __builtin_amdgcn_readfirstlane(max(0, min(16, Ltot - (t * kBN + group * 16))));
    const __amdgpu_buffer_rsrc_t rsrc =
        __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, base ? rows * (int)row_bytes : 0, 0x00020000);
#pragma unroll
    for (int k = 0; k < F::loads; ++k) lds_load_b128(rsrc, dst + k * kSeg, t_off[k]);
  };
  auto load_k_tile = [&](int t, int h) __attribute__((always_inline)) {
    issue_tile.template operator()<false>(lane_bcast((t >> 4) == win ? ak_cur : ak_nxt, ((t & 15) << 2) + group), t, dst_in(Ks, h, h + 1));
  };
  auto load_v_tile = [&](int t, int h) __attribute__((always_inline)) {
    issue_tile.template operator()<false>(lane_bcast((t >> 4) == win ? av_cur : av_nxt, ((t & 15) << 2) + group), t, dst_in(Vs, h, h + 1));
  };
  // Inside the main loop the same loads are split in two: the bases of the tiles an iteration will request
  // (K two tiles ahead, V one) are broadcast out of the windows during the iteration before, between its half-steps,
  // so that the iteration itself starts with nothing but its load instructions (four, eight with four wavefronts).  Right after a barrier every
  // wave of the workgroup is at this point at once, and what stands here keeps all matrix cores waiting.
  uint64_t nk = 0, nv = 0;
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
    const int tk = kt_next + 2, tv = kt_next + 1;   // (V's window is the current one)
    const int ik = ((tk & 15) << 2) + group;
    nk = (tk >> 4) == win ? lane_bcast(ak_cur, ik) : lane_bcast(ak_nxt, ik);
    nv = lane_bcast(av_cur, ((tv & 15) << 2) + group);
  };
  // a wave's direct loads are in LDS once its vector-memory counter has drained; the barrier then publishes them
  auto tile_barrier = [&]() __attribute__((always_inline)) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
  };

  // ---- the steps of the pipeline ----
  // Work advances in 32-key sub-tiles (half an LDS tile), three of them in flight: half-step h puts the scores of
  // sub-tile h + 1 and the output update with sub-tile h - 1 on the matrix core and computes the softmax of sub-tile
  // h on the vector ALU.  Nothing inside a half-step depends on anything else inside it, so its 32 MFMAs alternate
  // (two score, two output, two score, ...) with the vector instructions of a score pair between its two and those of an output pair
  // behind it: the vector work runs beside the MFMAs.  Two score accumulators and two P^T buffers alternate.
  // A fragment serves the two query groups: 16x16x32 takes the fragment reads and the cycles of 32x32x16 and moves half as much through
  // the accumulators, and the chip's clock under matrix load depends on what moves (skv_mfma_rate on N(0,1) operands 1865 -> 2125 TFLOP/s,
  // with an operand read and the least of this softmax beside each pair 1485 -> 1582).  Clock in this loop 1.70 -> 1.89 GHz, 64 requests of
  // 100 .. 9000 rows 14.0 -> 13.3 ms (1150 -> 1211 TFLOP/s), of 1070 791 -> 756 us.
  typedef f32x4 Scores[2][2];   // S^T of a sub-tile: [k][g][i]: key 16 k + 4 quad + i, query 16 g + l16; raw dot products
  Scores s[2];
  bf16x8 pb[2][2];  // P^T as B operands: [sub-tile parity][g], keys 4 quad .. + 3 and 16 + 4 quad .. + 3
  bf16x8 kfr[4];    // K fragment ring: runs four fragments ahead, across sub-tiles
  bf16x8 vfr[4];    // V^T fragment ring, likewise
  float m_ref[2] = {0.f, 0.f};   // reference the exponentials are taken against (score * scale * log2(e): exp2 units), per query
  float l_run[2] = {0.f, 0.f};   // running row sum over this lane's keys
#pragma unroll
  for (int k = 0; k < 8; ++k) s[k >> 2][(k >> 1) & 1][k & 1] = zero4;
#pragma unroll
  for (int e = 0; e < 8; ++e) pb[0][0][e] = pb[0][1][e] = pb[1][0][e] = pb[1][1][e] = (__bf16)0.f;
  // K fragment i = (k, ks): lane (l16, quad) wants key 16 k + l16 of the sub-tile, chunk 4 ks + quad.
  const int k_lane = (l16 >> 2) * kSeg + (l16 & 3) * 32 + (quad ^ turn(l16 >> 2)) * 8;
  // The PV A operand wants, per lane (d = 16 a + l16), the eight keys {4 quad + 0..3, 16 + 4 quad + 0..3}
  // of the sub-tile -- the keys this lane's P^T registers hold.  Each four come from one LDS
  // transpose load: within 16 lanes, lane i supplies the address of 4 consecutive d of key (i / 4) at d
  // offset 4 (i % 4) and receives d offset i of the four keys.  They lie in segment quad (second load: four
  // segments on); the lane's 8 bytes are piece lane % 2 of chunk 2 a + (lane % 4) / 2.
  const int v_lane = quad * kSeg + (l16 >> 2) * 32 + (((lane & 3) >> 1) ^ turn(quad)) * 8 + 4 * (lane & 1);
  const uint32_t k_base = lds_addr(Ks + k_lane), v_base[2] = {lds_addr(Vs + v_lane), lds_addr(Vs + (v_lane ^ 16))};   // of even and odd a
  auto k_frag = [&](uint32_t at, int i, int more = 0) __attribute__((always_inline)) {   // at + more: byte offset of the sub-tile
    return lds_read_b128(k_base + at, ((i >> 2) * 4 * kSeg + (i & 3) * 128) * 2 + more);
  };
  auto v_frag = [&](uint32_t at, int a, int more = 0) __attribute__((always_inline)) {
    const int off = (a >> 1) * 256 + more;
    const s16x4 lo = lds_read_tr16_b64(v_base[a & 1] + at, off);
    const s16x4 hi = lds_read_tr16_b64(v_base[a & 1] + at, off + 4 * kSeg * 2);
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
  };
  // causal mask of sub-tile u (keys 32 u ..), applied where the sub-tile reaches past the wave's first row
  auto mask = [&](Scores& x, int u) __attribute__((always_inline)) {
    const int key0 = u * 32;
    if (key0 + 31 > L + pos0) {
#pragma unroll
      for (int g = 0; g < 2; ++g) {
        const int limit = L + pos0 + ((16 * g + l16) >> hl_log);  // last visible key of this lane's query
#pragma unroll
        for (int e = 0; e < 8; ++e)
          if (key0 + (e >> 2) * 16 + quad * 4 + (e & 3) > limit) x[e >> 2][g][e & 3] = -INFINITY;
      }
    }
  };
  auto row_max = [&](const Scores& x, int g) __attribute__((always_inline)) {
    float m4[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) m4[k] = fmaxf(x[0][g][k], x[1][g][k]);
    return max_quads(fmaxf(fmaxf(m4[0], m4[1]), fmaxf(m4[2], m4[3])));
  };
  // Exponential k of a lane's sixteen: key group k / 8, query group (k / 4) % 2; plain fp32 adds for the row sum (the packed
  // dot-product instruction that would add a pair in one step does not run beside the MFMAs, the adds do).
  float ssum[2];
  auto arg = [&](const Scores& cur, int k) __attribute__((always_inline)) {
    const int g = (k >> 2) & 1;
    return __builtin_fmaf(cur[k >> 3][g][k & 3], c, -m_ref[g]);
  };
  auto pack = [&](int k, float e0, float e1, bf16x8 (&p_make)[2]) __attribute__((always_inline)) {   // pair k
    const f32x2 pr = {e0, e1};
    const bf16x2 cv = __builtin_convertvector(pr, bf16x2);
    const int at = (k >> 2) * 4 + 2 * (k & 1);
    p_make[(k >> 1) & 1][at] = cv[0];
    p_make[(k >> 1) & 1][at + 1] = cv[1];
  };
  auto tripped = [&]() __attribute__((always_inline)) { return __any(!(ssum[0] <= kSumLimit) || !(ssum[1] <= kSumLimit)); };
  auto exps = [&](const Scores& cur, bf16x8 (&p_make)[2]) __attribute__((always_inline)) {   // all of them
    ssum[0] = ssum[1] = 0.f;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const float e0 = __builtin_amdgcn_exp2f(arg(cur, 2 * k)), e1 = __builtin_amdgcn_exp2f(arg(cur, 2 * k + 1));
      pack(k, e0, e1, p_make);
      ssum[(k >> 1) & 1] += e0;
      ssum[(k >> 1) & 1] += e1;
    }
  };
  // The softmax keeps a reference per query; exponentials are taken against it as it stands, which leaves the
  // normalised result unchanged.  Only when a lane's sum of exponentials over a sub-tile passes kSumLimit (an element
  // at least kSumLimit / 8 above the reference; infinities and NaNs trip it too) is the reference moved to that
  // sub-tile's row maximum: O and the row sum are rescaled and this sub-tile's exponentials are taken again.  This
  // happens between half-steps, after the output update that still belongs to the old reference has been issued.
  auto move_reference = [&](const Scores& cur, bf16x8 (&p_make)[2]) __attribute__((always_inline)) {
#pragma unroll
    for (int g = 0; g < 2; ++g) {
      const float mx = row_max(cur, g) * c;
      const bool trip = !(max_quads(ssum[g]) <= kSumLimit);
      const float m_new = trip ? mx : m_ref[g];
      const float alpha = __builtin_amdgcn_exp2f(m_ref[g] - m_new);
      m_ref[g] = m_new;
      l_run[g] *= alpha;
#pragma unroll
      for (int a = 0; a < 8; ++a) o[a][g] *= alpha;
    }
    exps(cur, p_make);
  };
  auto active = [&](int u) __attribute__((always_inline)) { return u * 32 < wave_key_end; };
  // One half-step.  kb / kb_next: K of sub-tiles h + 1 and h + 2 (byte offsets in LDS); vb / vb_next: V of sub-tiles h - 1 and h.
  // The rings hold fragments 0..3 of sub-tile h + 1 (K) and of sub-tile h - 1 (V^T) on entry and are refilled behind
  // each MFMA with fragments 4..7 and then with fragments 0..3 of the following sub-tile.
  // Fast form (every stage at work, no masked key in sub-tile h): the 32 MFMAs alternate and carry the softmax between
  // them; a fragment is waited for four steps after its request, with the ten or eleven reads behind it outstanding.  kOff ..: constant parts of the four addresses.
  auto half_step_fast = [&]<bool kMask, int kOff = 0, int kOffNext = 0, int vOff = 0, int vOffNext = 0>(
                                        int h, uint32_t kb, uint32_t kb_next, uint32_t vb, uint32_t vb_next, Scores& dst,
                                        Scores& cur, bf16x8 (&p_use)[2], bf16x8 (&p_make)[2]) __attribute__((always_inline)) {
    if (kMask) mask(cur, h);
    ssum[0] = ssum[1] = 0.f;
    // One exponential behind the first MFMA of every pair (and one in front of them all), never two in a row: the transcendental
    // unit takes about four issue slots per instruction but works beside the issue port, so a second one right behind the
    // first would hold the wavefront until the unit is free again.  Its argument is worked out a pair ahead, for the same reason; a pair of
    // weights is packed and summed one step later; the last one comes a step early, so that the sums are there when the last MFMA has been
    // issued.  (Argument and exponential together behind the pair, one wait for both fragments: 1 to 3 % slower.)
    // The rest of a score pair's vector work stands between its MFMAs as well, and an output pair's second group goes first: 32 requests of
    // 256 .. 270 rows behind 25600 .. 25920 keys 3362 / 3335 us, 64 of 100 .. 9000 rows 13.06 / 13.01 ms, 1070 rows the same.  (The output
    // pair's work between its MFMAs too: 3387, 13.10.)
    float e[16], arg_next = arg(cur, 1);
    auto sum = [&](int k) __attribute__((always_inline)) { ssum[(k >> 2) & 1] += e[k]; };
    e[0] = __builtin_amdgcn_exp2f(arg(cur, 0));
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int k = i >> 2, ks = i & 3;
      lds_wait(11, kfr[i & 3]);   // behind it: its V^T fragment, three steps
      dst[k][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kfr[i & 3], qf[0][ks], ks == 0 ? zero4 : dst[k][0], 0, 0, 0);
      e[2 * i + 1] = __builtin_amdgcn_exp2f(arg_next);
      if (i < 7) arg_next = arg(cur, 2 * i + 2);
      if (i > 0) sum(2 * i - 2);
      dst[k][1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kfr[i & 3], qf[1][ks], ks == 0 ? zero4 : dst[k][1], 0, 0, 0);
      kfr[i & 3] = i < 4 ? k_frag(kb, i + 4, kOff) : k_frag(kb_next, i - 4, kOffNext);
      __builtin_amdgcn_sched_barrier(0);
      lds_wait(10, vfr[i & 3]);   // behind it: three steps, a K fragment
      o[i][1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vfr[i & 3], p_use[1], o[i][1], 0, 0, 0);
      if (i < 7) e[2 * i + 2] = __builtin_amdgcn_exp2f(arg_next);
      o[i][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vfr[i & 3], p_use[0], o[i][0], 0, 0, 0);
      vfr[i & 3] = i < 4 ? v_frag(vb, i + 4, vOff) : v_frag(vb_next, i - 4, vOffNext);
      if (i < 7) arg_next = arg(cur, 2 * i + 3);
      if (i > 0) {
        pack(i - 1, e[2 * i - 2], e[2 * i - 1], p_make);
        sum(2 * i - 1);
      }
      if (i == 7) {
        pack(7, e[14], e[15], p_make);
        sum(14);
        sum(15);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    if (__builtin_expect(tripped(), 0)) move_reference(cur, p_make);
    l_run[0] += ssum[0];
    l_run[1] += ssum[1];
  };
  // General form (first and last iterations of a wave): each stage is tested and runs as a block of its own; an MFMA waits
  // for its fragment with the three requested since behind it.
  auto half_step_slow = [&](int h, uint32_t kb, uint32_t kb_next, uint32_t vb, uint32_t vb_next, Scores& dst,
                            Scores& cur, bf16x8 (&p_use)[2], bf16x8 (&p_make)[2]) __attribute__((always_inline)) {
    if (active(h + 1)) {
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        lds_wait(3, kfr[i & 3]);
#pragma unroll
        for (int g = 0; g < 2; ++g)
          dst[i >> 2][g] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kfr[i & 3], qf[g][i & 3], (i & 3) == 0 ? zero4 : dst[i >> 2][g], 0, 0, 0);
        kfr[i & 3] = i < 4 ? k_frag(kb, i + 4) : k_frag(kb_next, i - 4);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    if (h > 0 && active(h - 1)) {
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        lds_wait(6, vfr[i & 3]);
#pragma unroll
        for (int g = 0; g < 2; ++g) o[i][g] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vfr[i & 3], p_use[g], o[i][g], 0, 0, 0);
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
      exps(cur, p_make);
      if (__builtin_expect(tripped(), 0)) move_reference(cur, p_make);
      l_run[0] += ssum[0];
      l_run[1] += ssum[1];
    }
    // whatever follows finds every fragment of the rings in place
    lds_wait(0, kfr[0], kfr[1], kfr[2], kfr[3]);
    lds_wait(0, vfr[0], vfr[1], vfr[2], vfr[3]);
  };

  // ---- prologue: tiles K(0), K(1), V(0); scores of sub-tile 0; the reference starts at its row maxima
  load_k_tile(0, 0);
  if (n_tiles > 1) load_k_tile(1, 2);
  load_v_tile(0, 0);
  stage_q();
  tile_barrier();
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    kfr[j] = k_frag(0, j);
    vfr[j] = kfr[j];   // defined; the V^T ring fills itself during half-step 0
  }
  if (active(0)) {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      lds_wait(3, kfr[i & 3]);
#pragma unroll
      for (int g = 0; g < 2; ++g)
        s[0][i >> 2][g] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kfr[i & 3], qf[g][i & 3], (i & 3) == 0 ? zero4 : s[0][i >> 2][g], 0, 0, 0);
      kfr[i & 3] = i < 4 ? k_frag(0, i + 4) : k_frag(0, i - 4, kHalfBytes);
      __builtin_amdgcn_sched_barrier(0);
    }
    // (idle states for the last MFMA: the compiler's wait-state insertion does not look through the branch inside
    // mask(), and the row maximum behind it would read score registers the matrix core has not written yet)
    asm volatile("s_nop 7\n\ts_nop 7\n\ts_nop 3" : "+v"(s[0][0][0]), "+v"(s[0][0][1]), "+v"(s[0][1][0]), "+v"(s[0][1][1]));
    mask(s[0], 0);
    // key 0 is visible to every query; finite also where its score and those of the other first keys are -infinity (the
    // reference then moves with the first score above it, and a part without any leaves nothing)
#pragma unroll
    for (int g = 0; g < 2; ++g) m_ref[g] = fmaxf(row_max(s[0], g) * c, -3.0e38f);
  }
  if (kTwo) __syncthreads();   // K's half 5, requested in iteration 0, takes the stage of half 0

  // ---- main loop.  Iteration kt (two half-steps) reads K(kt), K(kt + 1), V(kt - 1), V(kt).  It starts behind the
  // barrier that published K(kt + 1) and V(kt) and behind which no wave still reads K(kt - 1) or V(kt - 2): their
  // stages take the direct loads of K(kt + 2) and V(kt + 1), in flight during the whole iteration.  One barrier per
  // tile, none behind the last, and after it the output update with the last sub-tile (as an iteration of its own with its barrier,
  // and with the workgroup's place found by divisions, a work item of a tile took 9.2 us instead of 8: 512 requests of 64 rows
  // 164 -> 143 us, 64 of 1070 737 -> 722).
  // Iterations [1, kt_fast) of this wave have all three stages at work, no masked key and no ragged tile to load.
  // (told to be the same in all lanes: the compiler holds what it is not sure of in vector registers, four too many)
  const int kt_fast = __builtin_amdgcn_readfirstlane(min(min((L + pos0 - 63) / 64 + 1, (wave_key_end - 1) / 64), n_tiles - 3));
  // Iterations [kt_fast, kt_mid) still have all three stages at work in both half-steps, but keys may be masked and
  // the tiles they request may be ragged or absent (the last two or three before the diagonal tile): they run the
  // fast form with the mask applied and the general loads.
  const int kt_mid = (wave_key_end - 1) / 64;
  int h0 = 0;   // stage of K's half 2 kt and V's; half u sits in stage u % kHalves
  auto requests = [&]<bool kFast>(int kt, int h2, int h3, int h4, int h5) __attribute__((always_inline)) {   // stages of halves 2 kt + 2 ..
    if (__builtin_expect(pend, 0)) {
      window_bases(win + 1, pend_page, ak_nxt, av_nxt);
      pend = false;
    }
    if (kFast || kt + 2 < n_tiles) issue_tile.template operator()<kFast>(nk, kt + 2, dst_in(Ks, h4, h5));
    if (kFast || kt + 1 < n_tiles) issue_tile.template operator()<kFast>(nv, kt + 1, dst_in(Vs, h2, h3));
  };
  auto iteration = [&]<bool kMasked>(int kt) __attribute__((always_inline)) {   // general form, or the fast one with masks
    auto in = [&](int u) __attribute__((always_inline)) { return h0 + u >= kHalves ? h0 + u - kHalves : h0 + u; };   // of half 2 kt + u
    const int h1 = in(1), h2 = in(2), h3 = in(3), h_1 = in(kHalves - 1);
    requests.template operator()<false>(kt, h2, h3, in(4), in(5));
    const uint32_t k1 = h1 * kHalfBytes, k2 = h2 * kHalfBytes, k3 = h3 * kHalfBytes;                     // K
    const uint32_t v_1 = h_1 * kHalfBytes, v0 = h0 * kHalfBytes, v1 = h1 * kHalfBytes;                  // V
    if (kMasked) {
      half_step_fast.template operator()<true>(2 * kt, k1, k2, v_1, v0, s[1], s[0], pb[1], pb[0]);
      prep_bases(kt + 1);
      half_step_fast.template operator()<true>(2 * kt + 1, k2, k3, v0, v1, s[0], s[1], pb[0], pb[1]);
    } else {
      half_step_slow(2 * kt, k1, k2, v_1, v0, s[1], s[0], pb[1], pb[0]);
      prep_bases(kt + 1);
      half_step_slow(2 * kt + 1, k2, k3, v0, v1, s[0], s[1], pb[0], pb[1]);
    }
    if (kMasked || kt + 1 < n_tiles) tile_barrier();   // (nothing is published in the last one)
    h0 = h2;
  };
  // The fast form, unrolled until the stages repeat: they are constants and go into the reads' offset fields.
  auto fast = [&]<int kH>(int kt) __attribute__((always_inline)) {   // kH: h0
    constexpr int h1 = (kH + 1) % kHalves, h2 = (kH + 2) % kHalves, h3 = (kH + 3) % kHalves, h_1 = (kH + kHalves - 1) % kHalves;
    requests.template operator()<true>(kt, h2, h3, (kH + 4) % kHalves, (kH + 5) % kHalves);
    half_step_fast.template operator()<false, h1 * kHalfBytes, h2 * kHalfBytes, h_1 * kHalfBytes, kH * kHalfBytes>(2 * kt, 0, 0, 0, 0, s[1], s[0], pb[1], pb[0]);
    prep_bases(kt + 1);
    half_step_fast.template operator()<false, h2 * kHalfBytes, h3 * kHalfBytes, kH * kHalfBytes, h1 * kHalfBytes>(2 * kt + 1, 0, 0, 0, 0, s[0], s[1], pb[0], pb[1]);
    tile_barrier();
  };
  int kt = 0;
  prep_bases(0);
  iteration.template operator()<false>(kt++);
  // (of two workgroups the one whose items are short does without: it would take more than the 240 registers that leave the copy beside
  // them its 32)
  if constexpr (!kTwo) {
    for (; kt + 2 < kt_fast; kt += 3) {
      fast.template operator()<2>(kt);
      fast.template operator()<4>(kt + 1);
      fast.template operator()<0>(kt + 2);
    }
  }
  for (; kt < kt_mid; ++kt) iteration.template operator()<true>(kt);
  for (; kt < n_tiles; ++kt) iteration.template operator()<false>(kt);
  if (active(2 * n_tiles - 1)) {   // the output update with the last sub-tile
    const uint32_t vb = (h0 == 0 ? kHalves - 1 : h0 - 1) * kHalfBytes;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      if (i >= 4) lds_wait(14 - 2 * i, vfr[i & 3]);   // (0 .. 3 are there)
#pragma unroll
      for (int g = 0; g < 2; ++g) o[i][g] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vfr[i & 3], pb[1][g], o[i][g], 0, 0, 0);
      if (i < 4) vfr[i & 3] = v_frag(vb, i + 4);
      __builtin_amdgcn_sched_barrier(0);
    }
  }

  // ---- a part of a split item: O^T as it lies in the registers, the reference and the row sum
  if (pos0 >= row1) return;
  // (the lane number anew: what is addressed by it from here on would otherwise be worked out in front of the main loop and
  // hold registers through it)
  int lane_e;
  asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(lane_e));
  const int row_e = lane_e & 15, quad_e = lane_e >> 4;
  if (part) {
    const int slot = (part >> kPartBits) - 1;
    const int unit = kvh * n_hg + hg;
    f32x4* dst = (f32x4*)(p.partials + ((size_t)slot * p.Hkv * n_hg + unit) * kSlotFloats + (size_t)wave * (64 * 66)) + lane_e;
    float* const ml = (float*)(dst - lane_e + 16 * 64) + row_e;
#pragma unroll
    for (int g = 0; g < 2; ++g) {
      const float l_all = sum_quads(l_run[g]);
      if (pos0 + ((16 * g + row_e) >> hl_log) >= row1) continue;   // not a row of the tile: never read
#pragma unroll
      for (int a = 0; a < 8; ++a) dst[(a * 2 + g) * 64] = o[a][g];
      if (quad_e == 0) {
        ml[16 * g] = m_ref[g];
        ml[64 + 16 * g] = l_all;
      }
    }
    return;
  }

  if constexpr (kTwo) stage = Ks + ((h0 == 1 || h0 == 2) ? 2 * kHalf : 0) + wave * (kStageRows * kD);   // K's stages but half 2 n_tiles - 1, which others may still read
  // ---- normalise and store.  A lane holds queries l16 and 16 + l16 with d = 16 a + 4 quad + i, i.e. eight 8-byte
  // pieces of each one's output row.  They go through the wave's staging tile, 16 rows at a time, and leave as whole
  // 256-byte rows.
  {
    const int c16 = lane_e & 15;
#pragma unroll
    for (int pass = 0; pass < 2; ++pass) {
      const float inv = 1.0f / sum_quads(l_run[pass]);
      __bf16* const row = stage + row_e * kD;
#pragma unroll
      for (int a = 0; a < 8; ++a) {
        const f32x4 x = o[a][pass] * inv;
        const bf16x2 y0 = __builtin_convertvector(f32x2{x[0], x[1]}, bf16x2);
        const bf16x2 y1 = __builtin_convertvector(f32x2{x[2], x[3]}, bf16x2);
        const int chunk = 2 * a + (quad_e >> 1);   // its half quad % 2
        *(u32x2*)(row + (((chunk ^ row_e) << 3) + 4 * (quad_e & 1))) = u32x2{__builtin_bit_cast(uint32_t, y0), __builtin_bit_cast(uint32_t, y1)};
      }
      // same wave wrote and reads: the LDS operations of one wave complete in order
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int rr = (lane_e >> 4) + 4 * i;   // row within the pass
        const int pos = pos0 + ((16 * pass + rr) >> hl_log), head = head0 + (rr & ((1 << hl_log) - 1));
        const u32x4 v = *(const u32x4*)(stage + rr * kD + ((c16 ^ rr) << 3));
        if (pos < row1)   // (Q and the output pass once: they leave L2 to K and V)
          __builtin_nontemporal_store(v, (u32x4*)((__bf16*)p.out + ((size_t)(qbase + pos) * p.Hq + head) * kD + c16 * 8));
      }
    }
  }
}

// ---- merge of the parts of split items -----------------------------------------------------------
// One workgroup per (split item, kv head and head group, wavefront of the attention kernel); its wavefront q combines
// d = 32 (q % 4) .. + 31 of 16 of that wavefront's 32 rows, each lane what the same lane of every part wrote: coalesced 1 KB reads.
// Bound by latency: eight parts' states travel together and are folded into a running maximum, so the usual item takes one or
// two trips to memory (references first and outputs after them, four parts at a time: 10.7 us for 10 parts of 3 items,
// now 6.5).
constexpr int kMergeThreads = 512, kMergeParts = 8, kMergeGrid = 256;   // (most calls merge little or nothing)
__device__ __forceinline__ void merge_parts(const AttnParams& p, int n_blocks) {
  const int n_hg = p.Hq / p.Hkv / p.heads_per_wg, units = p.Hkv * n_hg;
  int rest, kvh, hg;
  unit_of_block(blockIdx.x, p.Hkv, n_hg, rest, kvh, hg);
  // (the record travels with the count: there is room for kCus of them, whatever the count)
  int4 a = ((const int4*)(p.splits + kSplitInts * min(rest / kWaves, kCus - 1)))[0];
  int parts = p.splits[kSplitInts * min(rest / kWaves, kCus - 1) + 4];
  const int n_work = p.n_items[1] * units * kWaves;
  for (int b = blockIdx.x; b < n_work; b += n_blocks) {
    if (b != (int)blockIdx.x) {
      unit_of_block(b, p.Hkv, n_hg, rest, kvh, hg);
      a = ((const int4*)(p.splits + kSplitInts * (rest / kWaves)))[0];
      parts = p.splits[kSplitInts * (rest / kWaves) + 4];
    }
    const int wave = rest % kWaves, unit = kvh * n_hg + hg;
    const int row0 = a.x, row1 = a.y, qbase = a.z, slot = a.w;
    const int lane = threadIdx.x & 63, q = threadIdx.x >> 6;
    const Packing pk = packing(p.heads_per_wg);
    int row, head;
    pk.wave(wave, row0, head, row);
    const int at = 16 * (q >> 2) + (lane & 15);   // of the 32 rows
    row += at >> pk.heads_log;
    if (row >= row1) continue;
    const size_t stride = (size_t)units * kSlotFloats;   // from one part to the next
    const float* src = p.partials + ((size_t)slot * units + unit) * kSlotFloats + (size_t)wave * (64 * 66);
    float m = -INFINITY, l = 0.f;
    f32x4 acc[2] = {};
    for (int j0 = 0; j0 < parts; j0 += kMergeParts) {   // (behind the end the last part stands in)
      float ms[kMergeParts], ls[kMergeParts], m_new = m;
      f32x4 x[kMergeParts][2];
#pragma unroll
      for (int k = 0; k < kMergeParts; ++k) {
        const float* s = src + min(j0 + k, parts - 1) * stride;
        ms[k] = s[64 * 64 + at];
        ls[k] = s[64 * 65 + at];
#pragma unroll
        for (int i = 0; i < 2; ++i) x[k][i] = ((const f32x4*)s)[((2 * (q & 3) + i) * 2 + (q >> 2)) * 64 + lane];
      }
#pragma unroll
      for (int k = 0; k < kMergeParts; ++k) m_new = fmaxf(m_new, ms[k]);
      const float keep = __builtin_amdgcn_exp2f(m - m_new);
      m = m_new;
      l *= keep;
#pragma unroll
      for (int i = 0; i < 2; ++i) acc[i] *= keep;
#pragma unroll
      for (int k = 0; k < kMergeParts; ++k) {
        if (j0 + k < parts) {
          const float w = __builtin_amdgcn_exp2f(ms[k] - m);
          l += w * ls[k];
#pragma unroll
          for (int i = 0; i < 2; ++i) acc[i] += w * x[k][i];
        }
      }
    }
    const float inv = 1.0f / l;
    head += kvh * (p.Hq / p.Hkv) + hg * p.heads_per_wg + (at & ((1 << pk.heads_log) - 1));
    __bf16* dst = (__bf16*)p.out + ((size_t)(qbase + row) * p.Hq + head) * kD + 32 * (q & 3) + 4 * (lane >> 4);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const bf16x2 y0 = __builtin_convertvector((f32x2{acc[i][0] * inv, acc[i][1] * inv}), bf16x2);
      const bf16x2 y1 = __builtin_convertvector((f32x2{acc[i][2] * inv, acc[i][3] * inv}), bf16x2);
      *(u32x2*)(dst + 16 * i) = u32x2{__builtin_bit_cast(uint32_t, y0), __builtin_bit_cast(uint32_t, y1)};
    }
  }
}

__global__ __launch_bounds__(kMergeThreads) void attn_merge_kernel(AttnParams p) { merge_parts(p, gridDim.x); }
// The merge waits for one read behind the other and the copy of a step's pages for the memory: where a step needs both they share
// a launch (merge_blocks workgroups, n_count for the counters of a request each, and the rest), two workgroups to a compute unit.  One request of 137 rows behind 2992 keys
// (187 pages): 8.0 + 7.0 us apart, 10.8 together.
__global__ __launch_bounds__(kMergeThreads, 4) void attn_merge_gather_kernel(AttnParams p, SkvGather g, SkvCount count, int merge_blocks, int n_count) {
  __shared__ int64_t first[kSkvGatherScan + 1];
  const int others = merge_blocks + n_count;
  if ((int)blockIdx.x < merge_blocks)
    merge_parts(p, merge_blocks);
  else if ((int)blockIdx.x < others)
    skv_count_request(count, (int)blockIdx.x - merge_blocks);
  else
    skv_gather_pages<true, true, kMergeThreads, 4>(g, (int)blockIdx.x - others, (int)gridDim.x - others, first, g.kpool, g.vpool,
                                                   g.matched_len, g.page_table, g.ctx_off, g.kctx, g.vctx);
}

// Query heads per workgroup: divides kWaves.  `fine`: eight where the kv head serves a multiple of eight.
int heads_per_wg_for(int G, bool fine) { return fine && G % 8 == 0 ? 8 : (G % 4 == 0 ? 4 : (G % 2 == 0 ? 2 : 1)); }

int check_attn(const skv_attn_desc* d) {
  if (!d) return SKV_EINVAL;
  if (d->n_q_heads < 1 || d->n_kv_heads < 1 || d->n_q_heads % d->n_kv_heads) return SKV_EINVAL;
  if (d->dtype == SKV_BF16) return d->head_dim == kD ? SKV_OK : SKV_EINVAL;
  if (d->dtype == SKV_F32) return (d->head_dim == 64 || d->head_dim == 128) ? SKV_OK : SKV_EINVAL;
  return SKV_EINVAL;
}

// How a call is laid out: from the description and the bounds the host knows.
struct Layout {
  bool two;                              // workgroups of four wavefronts, two to a compute unit
  int heads_per_wg, pos_log, units;      // pos_log: logarithm of the rows of a q tile; units: workgroups per item
  int64_t max_items, max_parts;          // max_parts: room for parts of split items, 0 if nothing is split
};
Layout layout_for(const skv_attn_desc* d, int32_t n_req, int64_t total_q_rows, bool fine, bool split, bool two = false) {
  Layout y;
  y.two = two;
  y.heads_per_wg = heads_per_wg_for(d->n_q_heads / d->n_kv_heads, fine);
  y.pos_log = kLogFull - two - __builtin_ctz(y.heads_per_wg);
  y.units = d->n_q_heads / y.heads_per_wg;
  y.max_parts = split && y.units <= kCus ? kMaxSlots / y.units : 0;
  y.max_items = (total_q_rows >> y.pos_log) + 2 * (int64_t)n_req + y.max_parts;   // per request: a short first tile and a ragged last one
  if (d->dtype != SKV_BF16) y.max_items = y.max_parts = 0;
  return y;
}
// What the host knows of a call: rows as if spread evenly, a table filled to its width.
int64_t mean_rows(int32_t n_req, int64_t total_q_rows) { return (total_q_rows + n_req - 1) / n_req; }
int64_t key_tiles(int64_t rows, int32_t max_blocks) { return ((int64_t)max_blocks * SKV_BLOCK_TOKENS + rows) / kBN + 1; }
// Whether any split can come of it (the device's rule, with items of 0.7 of the longest on average): where none can neither
// search nor merge are launched -- 3.2 us of a pass of 55.
bool may_split(const Layout& y, int32_t n_req, int64_t total_q_rows, int32_t max_blocks) {
  // more parts than there is room for
  if ((total_q_rows >> y.pos_log) * y.units > kMaxSlots || (int64_t)n_req * y.units > 2 * kMaxSlots) return false;
  const int64_t rows = mean_rows(n_req, total_q_rows), tiles = (rows + (1 << y.pos_log) - 1) >> y.pos_log, items = n_req * tiles;
  const float kt = (float)key_tiles(rows, max_blocks);
  const int last = tile_time((int)(rows - ((tiles - 1) << y.pos_log)), y.pos_log);
  const float share = 0.7f * n_req * y.units * ((tiles - 1) * kTileFull + last) * kt / kCus;
  return split_time(share, (float)total_q_rows / (items << y.pos_log)) <
         whole_time(items * y.units, kt * (tiles > 1 ? kTileFull : last), share);
}
// Whether workgroups find their items themselves (plan_item): a request per lane and, where items may be split, an item per
// lane, in one round of workgroups.  Behind the first round every workgroup, surplus ones too, would pay for it where a list is
// read in 1 us: 16 requests of 510 rows, 4.5 rounds, 497 us either way.
bool plan_in_place(const Layout& y, int32_t n_req) {
  const int64_t items = y.max_items - y.max_parts;
  return n_req <= kPlanRequests && items * y.units <= kCus && (!y.max_parts || items <= kPlanItems);
}
// Whether the parts of a split call are likely to be shorter in two rounds of workgroups, from what the host knows: such a call takes the list,
// whose kernel tries both.  Few items whose number does not divide a round: 3 requests of 770 rows behind 7.7 k cached tokens, 16 heads
// over 8, 21 items in 32 places stay whole in one round, 178 us, and are split in two, 134.  The list costs 5 us and the estimate
// errs where lengths differ, hence kTwoTiles (1986 calls of up to 14 requests behind up to 48 k: 0 / 10 / 16 / 30 tiles take the list for
// 253 / 159 / 115 / 72 of them; 83 / 80 / 67 / 46 are faster by 3 to 30 %, 108 / 37 / 20 / 8 slower by 3 to 9 %).
// The host does not see how uneven the lengths are, and two rounds take them better than one: the only request's are even, but of several
// whose longest part is kLongPart key tiles and more the list decides, at 4 % of such a call at most (372 of 14273 calls of 2 to 16
// requests take it for that, 112 faster by 3 to 37 %, 9 slower by 5 to 11: 2 of 351 and 377 rows behind 9.8 and 19 k, 64 heads over 8,
// 456 us in one round, 350; from 100 key tiles on twice the calls, and the rest of them no faster).
constexpr int kTwoTiles = 16, kLongPart = 150;
bool two_rounds(const Layout& y, int32_t n_req, int64_t total_q_rows, int32_t max_blocks) {
  const int64_t rows = mean_rows(n_req, total_q_rows), kt = key_tiles(rows, max_blocks);
  const int64_t items = n_req * ((rows + (1 << y.pos_log) - 1) >> y.pos_log);
  auto longest = [&](int64_t room) { return (kt + std::max<int64_t>(1, room / items) - 1) / std::max<int64_t>(1, room / items); };
  const int64_t one = longest(kCus / y.units);
  return (n_req > 1 && one >= kLongPart) || kStartTiles + one > 2 * (kStartTiles + longest(2 * kCus / y.units)) + kTwoTiles;
}
// Tiles of eight heads and 32 rows, or of four heads and 64: eight take half the workgroups for requests of up to 32 rows, and
// fewer where the last tile fits closer, but each costs half a key tile more (it may end inside one) and four heads in the one
// tile of a short request leave half the wavefronts idle, which makes a key tile shorter.  Where either fills the chip the sums decide,
// of requests that end anywhere in a tile: 64 query heads over 8, 256 requests of 1 .. 16 rows behind 500 to 1400 523 -> 322 us,
// 32 of 264 behind 16 .. 32 k 7.32 -> 6.83 ms.  Where four heads leave compute units without work eight would only leave more:
// one request of a row behind 512 15.8 us with four heads, 18.0 with eight; unless the keys are split, where the sums decide again
// (3 of a row behind 12000 64 -> 54 us).  A tile of up to 16 rows fills half the wavefronts of eight heads as well, one of up to 32 those
// of four: 15 requests of up to 6 rows behind up to 26 k, 64 over 8, 359 -> 216 us, 20 of a row behind 6 k 168 -> 89 (2573 shapes: other
// tiles for 121, their time 0.68 on average; 2 slower, by 5 and 8 %).  Splits from a list start later than the forecast's error allows
// for: they have to be a tenth shorter.
bool eight_heads(const skv_attn_desc* d, int32_t n_req, int64_t total_q_rows, int32_t max_blocks, bool split) {
  if ((d->n_q_heads / d->n_kv_heads) % 8) return false;
  const int64_t rows = mean_rows(n_req, total_q_rows);
  const float kt = (float)key_tiles(rows, max_blocks), at_ends = 6.f * kTileFull;   // at_ends: of a workgroup outside its loop
  const float tiles8 = std::max(1.f, rows / 32.f + 0.5f), tiles4 = std::max(1.f, rows / 64.f + 0.5f);
  const float wgs8 = (float)n_req * (d->n_q_heads / 8) * tiles8, wgs4 = (float)n_req * (d->n_q_heads / 4) * tiles4;
  const bool half8 = rows <= 16;
  const int tile8 = half8 ? kTileHalf : kTileFull;
  const float full = kt * kTileFull + at_ends, last4 = kt * (rows <= 32 ? kTileHalf : 0.5f * (kTileHalf + kTileFull)) + at_ends;
  const float whole8 = kt * tile8 + at_ends, time8 = wgs8 * (whole8 + (rows > 32 ? 0.5f * kTileFull : 0.f));
  const float time4 = (float)n_req * (d->n_q_heads / 4) * ((tiles4 - 1.f) * full + last4);
  if (wgs4 <= kCus) {
    if (!split) return false;
    if (rows > 32) return kt >= 32 && time8 < 0.98f * time4;
    const float most = half8 && !plan_in_place(layout_for(d, n_req, total_q_rows, true, true), n_req) ? 0.9f : 1.f;
    return split_time(wgs8 * kt * tile8 / kCus, (float)rows / kRowsPerWave) < most * whole_time(wgs4, kt * kTileHalf, 0.f);
  }
  return std::max(time8, kCus * whole8) < time4;
}
// Whether a call of whole items in several rounds takes workgroups of four wavefronts, two to a compute unit (tiles of half the rows,
// eight heads where the kv head serves a multiple of eight): one's start and end run under the other's loop, and in a tile of up to half
// the rows no wavefront is without any.  But K and V tiles travel twice as often: where items are long that counts for more, and where
// they fill one round nothing is gained.  us with one / two: 512 requests of 64 rows behind nothing 142 / 123, behind 512 keys 412 / 411;
// 1000 of 17 behind 32 177 / 98; 100 of 8 .. 32 behind 1600 .. 6400 339 / 309; 64 of 256 behind 8192 1956 / 2013; 8 query heads over 8, 64
// of 500 .. 1100 193 / 177; 24 over 8, 100 of 50 .. 100 104 / 72.  (1523 calls of 4 .. 400 requests of up to 800 rows behind up to 300
// pages: 0.87 of the time on average, 0.855 were every choice right; 48 are slower by 2 % and more, one by 16.  The width of the table and the
// mean rows are all that is known here, so lengths that differ and tables that are mostly empty are misjudged; the slower ones lie among the
// others: by heads, rows or workgroups every part of the calls is faster on average, eight heads in 400 to 450 workgroups, the worst, 0.96.)  Few rows behind
// kTwoPool and more of K and V: the copy of those pages, where a step makes one beside, is what takes the time, and the second set of loads
// costs it 2 to 3 % (128 of 8 .. 47 rows behind 2000 .. 3000, 1.5 GB: 550 / 566; 335 MB 130 / 130; 0.8 GB and 60 .. 105 rows 477 / 479).
constexpr int kTwoKeys = 25, kTwoKeysEight = 16;   // key tiles of an item in the middle of its request
constexpr float kTwoPool = 1 << 30;
bool two_workgroups(const skv_attn_desc* d, const Layout& z, int32_t n_req, int64_t total_q_rows, int32_t max_blocks) {
  const int64_t rows = mean_rows(n_req, total_q_rows), tile = 1 << z.pos_log;
  const float wgs = (float)n_req * z.units * std::max(1.f, (float)rows / (2 * tile) + 0.5f);
  const float keys = max_blocks * (float)SKV_BLOCK_TOKENS / kBN + rows / (2.f * kBN);
  if (wgs <= kCus || (rows > tile && keys > (z.heads_per_wg == 8 ? kTwoKeysEight : kTwoKeys))) return false;
  return rows > 2 * tile || (float)n_req * max_blocks * d->n_kv_heads * (SKV_BLOCK_TOKENS * kD * 4) < kTwoPool;
}
// Keys above which a longest request has the requests ordered by length.  Order is worth its 1.3 us where workgroups queue and
// one that starts late ends late: in a few rounds (64 requests of up to 39 rows behind up to 496, 16 query heads over 1: 42 ->
// 35 us), or behind long prefixes; many rounds of short requests run better as they come (200 of up to 63 rows, 32 over 8: 60.6 ->
// 55).
int order_above(const Layout& y, int32_t n_req, int64_t total_q_rows) {
  const float tiles = std::max(1.f, (float)mean_rows(n_req, total_q_rows) / (1 << y.pos_log) + 0.5f), wgs = tiles * n_req * y.units;
  return wgs <= kCus ? INT_MAX : wgs <= 4 * kCus ? 0 : 1024;
}
size_t split_bytes(const Layout& y) {
  return y.max_parts ? kCus * kSplitInts * sizeof(int32_t) + (size_t)y.max_parts * y.units * kSlotFloats * sizeof(float) : 0;
}

size_t list_offset(const skv_attn_desc* d) {
  return 256 + (d->dtype == SKV_BF16 ? skv_align256((size_t)SKV_BLOCK_TOKENS * d->n_kv_heads * kD * 2) : 0);
}

}  // namespace

// What a call needs at the least: the work list, behind a page that no kernel uses any longer and that the interface's sizes (what
// is accepted, what is refused) go on to count.  The size does not fall as n_req or total_q_rows grow.
static size_t list_bytes(const skv_attn_desc* d, const Layout& y) {
  return list_offset(d) + skv_align256((size_t)y.max_items * kItemInts * sizeof(int32_t));
}

extern "C" int skv_prefill_attn_workspace_size(const skv_attn_desc* desc, int32_t n_req,
                                               int64_t total_q_rows, size_t* bytes) {
  int rc = check_attn(desc);
  if (rc) return rc;
  if (n_req < 0 || total_q_rows < 0 || !bytes) return SKV_EINVAL;
  *bytes = 0;
  for (const bool fine : {false, true}) {   // whichever tiles a call takes
    const Layout y = layout_for(desc, n_req, total_q_rows, fine, true);
    *bytes = std::max(*bytes, list_bytes(desc, y) + split_bytes(y));
  }
  return SKV_OK;
}

// The layout of a call that splits nothing, with list_room bytes for the list.  Where none fits it is the smallest, for the caller to refuse.
static bool too_many_items(const skv_attn_desc* d, const Layout& y);
static Layout whole_layout(const skv_attn_desc* d, int32_t n_req, int64_t total_q_rows, int32_t max_blocks, size_t list_room) {
  Layout y = layout_for(d, n_req, total_q_rows, eight_heads(d, n_req, total_q_rows, max_blocks, false), false);
  if (list_bytes(d, y) > list_room) y = layout_for(d, n_req, total_q_rows, false, false);
  const Layout z = layout_for(d, n_req, total_q_rows, true, false, true);
  if (d->dtype == SKV_BF16 && !plan_in_place(y, n_req) && two_workgroups(d, z, n_req, total_q_rows, max_blocks) && list_bytes(d, z) <= list_room &&
      !too_many_items(d, z))
    y = z;
  return y;
}

// (fp32 has no list, and a limit of its own)
static bool too_many_items(const skv_attn_desc* d, const Layout& y) {
  return d->dtype == SKV_BF16 && (y.max_items * y.units > 0x7fffffff || y.max_items > 0x3fffffff);
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

// What a whole step behind its lookup adds: the suffix offsets, made from req_off, the gather, and counters the lookup left.
struct StepExtras {
  const int32_t* req_off;
  int32_t* q_off;
  SkvGather gather;
  SkvCount count;
};

// Shared by the entry points: enqueues the schedule kernel and the attention kernel on checked arguments.
static int prefill_attn_enqueue(const skv_attn_desc* desc, int32_t n_req, const void* d_q,
                                const void* d_knew, const void* d_vnew, const int32_t* d_q_off,
                                int64_t total_q_rows, const void* d_kpool, const void* d_vpool,
                                int32_t n_pages, const int32_t* d_matched_len,
                                const int32_t* d_page_table, int32_t max_blocks, void* d_out,
                                void* d_workspace, const Layout& y, const StepExtras* x, void* stream) {
  hipStream_t st = (hipStream_t)stream;
  // of up to kSkvGatherScan requests a plan with parts makes the suffix offsets itself, and its pages travel beside the merge
  const bool plan = desc->dtype == SKV_BF16 && !y.two && plan_in_place(y, n_req) && !(y.max_parts && two_rounds(y, n_req, total_q_rows, max_blocks));
  const bool late = x && plan && y.max_parts && !x->gather.large;
  if (x && !late && desc->dtype == SKV_BF16) {
    const int rc = skv_gather_enqueue(x->gather, false, x->req_off, x->q_off, x->count, stream);
    if (rc) return rc;
  }

  AttnParams p;
  p.q = d_q; p.knew = d_knew; p.vnew = d_vnew; p.kpool = d_kpool; p.vpool = d_vpool; p.out = d_out;
  p.page_table = d_page_table;
  p.n_items = (const int32_t*)d_workspace;
  p.items = (const int32_t*)((char*)d_workspace + list_offset(desc));
  p.max_blocks = max_blocks; p.n_pages = n_pages;
  p.Hq = desc->n_q_heads; p.Hkv = desc->n_kv_heads;
  p.heads_per_wg = y.heads_per_wg;
  p.G = p.Hq / p.Hkv;
  p.n_hg = p.G / y.heads_per_wg;
  p.scale = skv_softmax_scale(desc);

  if (desc->dtype == SKV_F32) {
    const SkvAttnF32Params f = {d_q, d_knew, d_vnew, d_kpool, d_vpool, d_out, d_q_off, d_matched_len, d_page_table,
                                n_req, max_blocks, n_pages, desc->n_q_heads, desc->n_kv_heads, skv_softmax_scale(desc),
                                total_q_rows, nullptr};
    const SkvStepRest rest = x ? SkvStepRest{&x->gather, x->req_off, x->q_off, &x->count} : SkvStepRest{};
    return skv_attn_f32_enqueue(f, desc->head_dim, x ? &rest : nullptr, stream);
  }

  // the list holds whole items or, where anything is split, no more than max_parts records
  const int64_t grid = (plan && y.max_parts ? kCus / y.units : std::max(y.max_items - y.max_parts, y.max_parts)) * y.units;
  char* const split_area = (char*)d_workspace + list_bytes(desc, y);
  p.splits = y.max_parts ? (const int32_t*)split_area : nullptr;
  p.partials = y.max_parts ? (float*)(split_area + kCus * kSplitInts * sizeof(int32_t)) : nullptr;
  p.q_off = d_q_off;
  p.matched_len = d_matched_len;
  p.req_off = late ? x->req_off : nullptr;
  p.q_off_out = late ? x->q_off : nullptr;
  p.n_items_out = (int32_t*)d_workspace;
  p.splits_out = (int32_t*)p.splits;
  p.n_req = n_req;
  p.pos_log = y.pos_log;
  p.max_items = (int)y.max_items;
  p.rows_filled = (float)total_q_rows * y.heads_per_wg;
  if (!plan) {
    attn_schedule_kernel<<<1, kSchedThreads, 0, st>>>(n_req, d_q_off, d_matched_len, y.pos_log, p.max_items, y.units,
                                                      order_above(y, n_req, total_q_rows), p.rows_filled, p.n_items_out, (int32_t*)p.items, p.splits_out);
    SKV_HIP(hipGetLastError());
  }
  const auto kernel = y.two ? attn_bf16_kernel<false, false, true>
                      : y.max_parts ? (plan ? attn_bf16_kernel<true, true, false> : attn_bf16_kernel<true, false, false>)
                                    : (plan ? attn_bf16_kernel<false, true, false> : attn_bf16_kernel<false, false, false>);
  kernel<<<(int)grid, y.two ? Form<true>::threads : kThreads, 0, st>>>(p);
  SKV_HIP(hipGetLastError());
  if (y.max_parts) {   // a split item has two parts at least
    const int merge_blocks = (int)std::min<int64_t>(y.max_parts / 2 * y.units * kWaves, kMergeGrid);
    const int n_count = late && x->count.records ? n_req : 0;
    if (late)
      attn_merge_gather_kernel<<<merge_blocks + n_count + skv_gather_blocks(x->gather), kMergeThreads, 0, st>>>(p, x->gather, x->count,
                                                                                                               merge_blocks, n_count);
    else
      attn_merge_kernel<<<merge_blocks, kMergeThreads, 0, st>>>(p);
    SKV_HIP(hipGetLastError());
  }
  return SKV_OK;
}

// Arguments checked and the layout chosen; y's list fits the workspace.  *empty: nothing to compute.
static int prefill_attn_check(const skv_attn_desc* desc, int32_t n_req, const void* d_q, const void* d_knew, const void* d_vnew,
                              const int32_t* d_q_off, int64_t total_q_rows, const void* d_kpool, const void* d_vpool, int32_t n_pages,
                              const int32_t* d_matched_len, const int32_t* d_page_table, int32_t max_blocks, const void* d_out,
                              const void* d_workspace, size_t workspace_bytes, Layout& y, bool& empty) {
  int rc = check_attn(desc);
  if (rc) return rc;
  if (n_req < 0 || total_q_rows < 0 || n_pages < 0 || max_blocks < 0) return SKV_EINVAL;
  empty = n_req == 0 || total_q_rows == 0;
  if (empty) return SKV_OK;
  rc = check_attn_buffers(d_q, d_knew, d_vnew, d_q_off, d_kpool, d_vpool, d_matched_len, d_page_table, max_blocks,
                          d_out);
  if (rc) return rc;
  // a workspace that holds the plain work list is enough: the call then splits nothing, and takes 32-row tiles if their list fits
  y = layout_for(desc, n_req, total_q_rows, eight_heads(desc, n_req, total_q_rows, max_blocks, true), true);
  if (!y.max_parts || !may_split(y, n_req, total_q_rows, max_blocks) || workspace_bytes < list_bytes(desc, y) + split_bytes(y))
    y = whole_layout(desc, n_req, total_q_rows, max_blocks, workspace_bytes);
  if (!d_workspace || workspace_bytes < list_bytes(desc, y)) return SKV_ENOMEM;
  if ((uintptr_t)d_workspace & 15) return SKV_EINVAL;
  return too_many_items(desc, y) ? SKV_ERANGE : SKV_OK;
}

extern "C" int skv_prefill_attn(const skv_attn_desc* desc, int32_t n_req, const void* d_q,
                                const void* d_knew, const void* d_vnew, const int32_t* d_q_off,
                                int64_t total_q_rows, const void* d_kpool, const void* d_vpool,
                                int32_t n_pages, const int32_t* d_matched_len,
                                const int32_t* d_page_table, int32_t max_blocks, void* d_out,
                                void* d_workspace, size_t workspace_bytes, void* stream) {
  Layout y;
  bool empty;
  const int rc = prefill_attn_check(desc, n_req, d_q, d_knew, d_vnew, d_q_off, total_q_rows, d_kpool, d_vpool, n_pages, d_matched_len,
                                    d_page_table, max_blocks, d_out, d_workspace, workspace_bytes, y, empty);
  if (rc || empty) return rc;
  return prefill_attn_enqueue(desc, n_req, d_q, d_knew, d_vnew, d_q_off, total_q_rows, d_kpool, d_vpool, n_pages,
                              d_matched_len, d_page_table, max_blocks, d_out, d_workspace, y, nullptr, stream);
}

extern "C" int skv_prefill_step(const skv_attn_desc* desc, int32_t n_req, const int32_t* d_req_off, const void* d_q,
                                const void* d_knew, const void* d_vnew, int32_t* d_q_off, int64_t total_q_rows,
                                const void* d_kpool, const void* d_vpool, int32_t n_pages, const int32_t* d_matched_len,
                                const int32_t* d_page_table, int32_t max_blocks, void* d_out, int64_t* d_ctx_off, void* d_kctx,
                                void* d_vctx, int64_t ctx_capacity_tokens, const skv_tree* tree, const int32_t* d_req_tenant,
                                const int32_t* d_records, void* d_workspace, size_t workspace_bytes, void* stream) {
  StepExtras x = {d_req_off, d_q_off, {}, {}};
  if (d_records) {
    if (!tree || !d_req_tenant || n_req < 0 || max_blocks < 0 || (n_req > 0 && !d_matched_len)) return SKV_EINVAL;   // nothing to count by
    x.count = {tree->dev.ctr, tree->dev.ctr_plane, d_records, d_req_tenant, d_matched_len, max_blocks, n_req};
  }
  int rc = SKV_EINVAL;
  if (n_req >= 0 && d_q_off && (n_req == 0 || (d_req_off && d_matched_len)))
    rc = skv_gather_check(desc, n_req, d_kpool, d_vpool, n_pages, d_matched_len, d_page_table, max_blocks, d_ctx_off, d_kctx, d_vctx,
                          ctx_capacity_tokens, &x.gather);
  if (rc) {   // (the lookup has happened: its counters are not lost)
    const int rn = skv_count_enqueue(x.count, stream);
    return rn ? rn : rc;
  }
  Layout y;
  bool empty = false;
  rc = prefill_attn_check(desc, n_req, d_q, d_knew, d_vnew, d_q_off, total_q_rows, d_kpool, d_vpool, n_pages, d_matched_len,
                          d_page_table, max_blocks, d_out, d_workspace, workspace_bytes, y, empty);
  if (rc || empty) {   // what does not depend on the attention happens all the same
    const int rg = skv_gather_enqueue(x.gather, false, d_req_off, d_q_off, x.count, stream);
    return rg ? rg : rc;
  }
  return prefill_attn_enqueue(desc, n_req, d_q, d_knew, d_vnew, d_q_off, total_q_rows, d_kpool, d_vpool, n_pages,
                              d_matched_len, d_page_table, max_blocks, d_out, d_workspace, y, &x, stream);
}

// ---- the same call for callers that cannot allocate ---------------------------------------------
// The work list lives in a file-scope device array instead of a caller workspace.  Every GPU
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
  const Layout y = whole_layout(desc, n_req, total_q_rows, max_blocks, SKV_STATIC_SCRATCH_BYTES);
  if (list_bytes(desc, y) > (size_t)SKV_STATIC_SCRATCH_BYTES || too_many_items(desc, y)) return SKV_ERANGE;   // batch too large for the built-in scratch
  void* ws = nullptr;
  rc = scratch_of_current_device(&ws);
  if (rc) return rc;
  // the schedule kernel rewrites the item count and every record it hands out on each call,
  // so nothing of the previous call's contents is read
  return prefill_attn_enqueue(desc, n_req, d_q, d_knew, d_vnew, d_q_off, total_q_rows, d_kpool, d_vpool, n_pages,
                              d_matched_len, d_page_table, max_blocks, d_out, ws, y, nullptr, stream);
}

// ---- measurement aid: what the matrix cores sustain on given operand values ----
// The clock the chip holds under matrix load depends on the values flowing through the multipliers, so the rate a
// kernel can reach is a property of its data as well as of its code.  Every wavefront keeps six (A, B) operand
// pairs of the caller's data in registers and issues the attention kernel's 16x16x32 MFMAs, an A operand with two B operands as there,
// back to back into eight pairs of accumulators: no memory traffic, no other instructions.  One workgroup of eight wavefronts per compute unit; its
// LDS claim keeps a second workgroup off the unit, so every SIMD runs exactly two wavefronts from start to end.
// With side work, every pair of MFMAs is accompanied by what the attention kernel's softmax issues per pair at the least --
// its A operand read from LDS (16 bytes per lane), one multiply-add, one exponential, one add and half a packed
// conversion -- on values that depend on nothing the matrix core produces: no dependency on a result, no global
// load, no barrier.  What this form sustains is a measure of that instruction mix, in the attention kernel's order.
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
  f32x4 c[8][2];
#pragma unroll
  for (int j = 0; j < 8; ++j) c[j][0] = c[j][1] = f32x4{0.f, 0.f, 0.f, 0.f};
  float t = 0.f;
  if (kSide) {
    // the workgroup's own 96 KB of operand data fill the LDS; a wavefront reads A operands from its own 8 KB of it
    constexpr int kVecs = kRateLdsBytes / 16;
    for (int i = threadIdx.x; i < kVecs; i += kRateThreads) claim[i] = ops[(size_t)blockIdx.x * kVecs + i];
    __syncthreads();
    const uint32_t abase = lds_addr(&claim[(threadIdx.x & 63) + (threadIdx.x >> 6) * 512]);
    bf16x8 ar[4] = {a[0], a[1], a[2], a[3]};   // ring: the read behind pair j serves pair j + 4
    float x[4], e_prev = 0.f, e_pp = 0.f;
#pragma unroll
    for (int j = 0; j < 4; ++j) x[j] = (float)((threadIdx.x * 37 + j * 101) % 1000) * 0.001f;
    for (int it = 0; it < iters; ++it) {
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        lds_wait(3, ar[j & 3]);
        c[j & 7][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ar[j & 3], b[(j / 4 + j) % kRatePairs], c[j & 7][0], 0, 0, 0);
        x[j & 3] = __builtin_fmaf(-1.9371f, __builtin_fabsf(x[j & 3]), 1.0f);   // bounded, never settles
        const float e = __builtin_amdgcn_exp2f(x[j & 3]);
        c[j & 7][1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ar[j & 3], b[(j / 4 + j + 3) % kRatePairs], c[j & 7][1], 0, 0, 0);
        ar[j & 3] = lds_read_b128(abase, (j & 7) * 1024);
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
#pragma unroll
        for (int g = 0; g < 2; ++g)
          c[j & 7][g] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[j % kRatePairs], b[(j / 4 + j + 3 * g) % kRatePairs], c[j & 7][g], 0, 0, 0);
    }
  }
#pragma unroll
  for (int j = 0; j < 16; ++j)
#pragma unroll
    for (int e = 0; e < 4; ++e) t += c[j >> 1][j & 1][e];
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
  if (flops) *flops = (double)blocks * (kRateThreads / 64) * (double)iters * 32.0 * (2.0 * 16 * 16 * 32);
  return SKV_OK;
}
