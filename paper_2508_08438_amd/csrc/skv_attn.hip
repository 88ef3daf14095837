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
// The rest of a step in the attention's launch: its pages and n_count requests' counters.  Needs nothing of the attention.
struct Rest {
  SkvGather gather;
  SkvCount count;
  int n_count, n_attn;   // n_attn: workgroups of the attention, in front
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

// kOffsets: q_off is still to come, it is made from req_off here (q_off_out).
template <bool kOffsets>
__global__ __launch_bounds__(kSchedThreads) void attn_schedule_kernel(
    int n_req, const int32_t* __restrict__ q_off /* or req_off */, int32_t* __restrict__ q_off_out, const int32_t* __restrict__ matched_len, int pos_log, int max_items,
    int units /* workgroups per item */, int order_above /* requests are ordered by length if one is longer */,
    float rows_filled /* query rows, over the heads of a workgroup */,
    int32_t* __restrict__ n_items /* [0] items, [1] split items */, int32_t* __restrict__ items, int32_t* __restrict__ splits /* null: never split */) {
  __shared__ int scan[kSchedThreads], red[kSchedWaves], bucket[kBuckets];
  __shared__ int4 req_at[kSchedThreads];   // request, first row, rows, reused length
  __shared__ int4 item_a[kCus], item_b[kCus];   // the first records, for the split
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int listed = 0, rows_before = 0;
  if (kOffsets && tid == 0) q_off_out[0] = 0;
  for (int base = 0; base < n_req; base += kSchedThreads) {
    const int r = base + tid, n_here = min(kSchedThreads, n_req - base);
    Cut mine = {};
    if constexpr (kOffsets) {
      const int matched = r < n_req ? matched_len[r] : 0, own = r < n_req ? max(0, q_off[r + 1] - q_off[r] - matched) : 0;
      int total;
      const int end = rows_before + skv_block_scan<kSchedThreads>(own, red, total);
      rows_before += total;
      if (r < n_req) {
        q_off_out[r + 1] = end;
        mine = cut_of(end - own, end, matched, pos_log);
      }
    } else if (r < n_req) {
      mine = cut_of(q_off[r], q_off[r + 1], matched_len[r], pos_log);
    }
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
// (The text is a file of its own for two kernels to hold: as a function of either it takes ten registers more, and the copy beside it no longer fits.)
template <bool kParts, bool kPlan, bool kTwo>
__global__ __launch_bounds__(Form<kTwo>::threads, 2) void attn_bf16_kernel(AttnParams p) {
#include "skv_attn_bf16.h"
}
// The same, and behind its workgroups those of the rest of a step.
template <bool kParts, bool kPlan, bool kTwo>
__global__ __launch_bounds__(Form<kTwo>::threads, 2) void attn_rest_kernel(AttnParams p, Rest x) {
  if ((int)blockIdx.x >= x.n_attn) {
    const int b = (int)blockIdx.x - x.n_attn;
    const SkvGather& g = x.gather;
    if (b < x.n_count) return skv_count_request(x.count, b);
    return skv_copy_pages<Form<kTwo>::threads, 4>(g.n_req, (const char*)g.kpool, (const char*)g.vpool, g.n_pages, g.matched_len, g.page_table,
                                                  g.max_blocks, g.ctx_off, (char*)g.kctx, (char*)g.vctx, g.cap_pages, g.page_vec * 16,
                                                  b - x.n_count, (int)gridDim.x - x.n_attn - x.n_count);
  }
#include "skv_attn_bf16.h"
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
bool forecast_splits(const Layout& y, int32_t n_req, int64_t total_q_rows, int32_t max_blocks, float mean) {   // mean: item to the longest
  const int64_t rows = mean_rows(n_req, total_q_rows), tiles = (rows + (1 << y.pos_log) - 1) >> y.pos_log, items = n_req * tiles;
  const float kt = (float)key_tiles(rows, max_blocks);
  const int last = tile_time((int)(rows - ((tiles - 1) << y.pos_log)), y.pos_log);
  const float share = mean * n_req * y.units * ((tiles - 1) * kTileFull + last) * kt / kCus;
  return split_time(share, (float)total_q_rows / (items << y.pos_log)) <
         whole_time(items * y.units, kt * (tiles > 1 ? kTileFull : last), share);
}
bool may_split(const Layout& y, int32_t n_req, int64_t total_q_rows, int32_t max_blocks) {
  // more parts than there is room for
  if ((total_q_rows >> y.pos_log) * y.units > kMaxSlots || (int64_t)n_req * y.units > 2 * kMaxSlots) return false;
  return forecast_splits(y, n_req, total_q_rows, max_blocks, 0.7f);
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

// Whether the rest of a step rides with its attention.  The copy and the counters need nothing of it, and the suffix offsets are made where the items
// are; behind its workgroups they fill the places that the last long ones leave, and a launch in front is saved.  us a pass, in front / so: 12
// requests of 100 .. 300 rows behind 300 .. 700 keys 61.4 / 51.3, 24 of 50 .. 150 98.0 / 88.8, 10 of 10 .. 60 with 64 heads 55.2 / 43.7.  The other
// arguments cost every workgroup 0.1 us of its start, so not in many rounds of them: of several hundred steps each 0.77 to 0.92 of the time in up to
// two rounds, 0.93 to 0.95 in two to five, 0.97 in six to twelve, 1.00 in twenty and more (64 of 1070 rows, 34 rounds, 743 either way). Nor where the
// copy is long and few rows leave it nothing to hide behind: there it has one workgroup to a compute unit at the most, and none of small pages keeps
// enough in flight.  Workgroups of four wavefronts: 613 pages of 32 KB, 63 requests of 3 rows, 28.2 / 32.8, 1416 of 84 of 29 62.7 / 69.9; up to 12 MB
// a pool 0.77 to 0.97; behind more than 128 rows 0.95 to 1.01 whatever its size.  Of eight, pages of 4 KB: 28.7 k of 121 of 2 rows 134 / 161, 5670 of
// 189 of 12 36.9 / 41.3, 58.6 k of 243 of up to 2 230 / 296; up to 16 MB 0.82 to 0.93, behind more than 128 rows 0.95 (the slowest 1.04).  Of eight,
// pages of 16 KB and more, 0.75 to 1.00 (large copies, which do not ride, 0.83 to 1.01). 4200 steps, other ones than these lines were drawn from:
// 0.93 of the time in front, 2 slower by 5 % and more (by 5 and 7), 76 without these limits and kRideWhole's (55 of them by 10 to 23).
constexpr int kRideRounds = 4, kRideRows = 128;
constexpr int64_t kRideTwo = 12 << 20, kRideSmall = 16 << 20;
static bool rest_rides(const SkvGather& g, const Layout& y, int64_t grid, int64_t rows) {   // rows: of a request
  if (y.units == 0 || y.max_items == 0 || g.n_req > kSkvGatherScan || g.large || (int64_t)g.page_vec * 16 > 0x7fffffff) return false;
  if (grid > kRideRounds * kCus * (y.two ? 2 : 1)) return false;
  const int64_t page_bytes = (int64_t)g.page_vec * 16, bytes = std::min((int64_t)g.n_req * g.max_blocks, g.cap_pages) * page_bytes;
  return rows > kRideRows || bytes < (y.two ? kRideTwo : page_bytes < 16384 ? kRideSmall : INT64_MAX);
}

// Whether it does so, too, where workgroups may split items in place, or shares the launch of the merge.  With the attention the copy fills what is
// idle but slows the parts, whose end is everybody's; beside the merge it takes time of its own.  So with long parts, and where long items are likely
// to stay whole, so that the merge has nothing to do.  us a pass, beside the merge / with the attention: 1 request of 256 rows behind 24 k keys, 64
// heads, parts of 126 key tiles 233 / 222; 900 rows behind 19 k, 164 tiles 296 / 282.  Parts, time with the attention to that beside the merge: of up
// to 10 tiles 1.01 to 1.11, the slowest 1.33, of 10 to 20 1.00 to 1.08, of 20 to 40 1.00 to 1.04, of 40 to 60 0.98 to 1.02, of 60 to 100 0.94 to
// 1.01, the slowest 1.08, from 100 on 0.92 to 1.01 (all the slower the larger the copy).  Whole items, 4 of 118 behind 2.2 k, 46 tiles, 103 / 88; of
// 40 tiles and more 0.92, the slowest 1.01; of 20 to 40 0.96, but where lengths differ parts come of it all the same and one in five is slower, 13 of
// 2 rows behind 800 .. 1600 40.6 / 46.3, 11 of 30 behind 1200 .. 2300, 37 tiles, 52.8 / 56.3.
constexpr int kRidePart = 100, kRideWhole = 40;
static bool rides_with_parts(const Layout& y, int32_t n_req, int64_t total_q_rows, int32_t max_blocks) {
  const int64_t rows = mean_rows(n_req, total_q_rows), kt = key_tiles(rows, max_blocks);
  const int64_t items = n_req * ((rows + (1 << y.pos_log) - 1) >> y.pos_log);
  return kt >= kRidePart * std::max<int64_t>(1, kCus / y.units / items) ||
         (kt >= kRideWhole && !forecast_splits(y, n_req, total_q_rows, max_blocks, 1.f));
}

// Shared by the entry points: enqueues the schedule kernel and the attention kernel on checked arguments.
static int prefill_attn_enqueue(const skv_attn_desc* desc, int32_t n_req, const void* d_q,
                                const void* d_knew, const void* d_vnew, const int32_t* d_q_off,
                                int64_t total_q_rows, const void* d_kpool, const void* d_vpool,
                                int32_t n_pages, const int32_t* d_matched_len,
                                const int32_t* d_page_table, int32_t max_blocks, void* d_out,
                                void* d_workspace, const Layout& y, const StepExtras* x, void* stream) {
  hipStream_t st = (hipStream_t)stream;
  // of up to kSkvGatherScan requests a plan with parts makes the suffix offsets itself, and its pages travel beside the merge where
  // they do not with the attention
  const bool plan = desc->dtype == SKV_BF16 && !y.two && plan_in_place(y, n_req) && !(y.max_parts && two_rounds(y, n_req, total_q_rows, max_blocks));
  const bool parts = plan && y.max_parts;
  // the list holds whole items or, where anything is split, no more than max_parts records
  const int64_t grid = (parts ? kCus / y.units : std::max(y.max_items - y.max_parts, y.max_parts)) * y.units;
  const bool ride = x && rest_rides(x->gather, y, grid, mean_rows(n_req, total_q_rows)) && (!parts || rides_with_parts(y, n_req, total_q_rows, max_blocks));
  const bool late = x && parts && !ride && !x->gather.large;
  if (x && !late && !ride && desc->dtype == SKV_BF16) {
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

  char* const split_area = (char*)d_workspace + list_bytes(desc, y);
  p.splits = y.max_parts ? (const int32_t*)split_area : nullptr;
  p.partials = y.max_parts ? (float*)(split_area + kCus * kSplitInts * sizeof(int32_t)) : nullptr;
  p.q_off = d_q_off;
  p.matched_len = d_matched_len;
  p.req_off = late || ride ? x->req_off : nullptr;
  p.q_off_out = late || ride ? x->q_off : nullptr;
  p.n_items_out = (int32_t*)d_workspace;
  p.splits_out = (int32_t*)p.splits;
  p.n_req = n_req;
  p.pos_log = y.pos_log;
  p.max_items = (int)y.max_items;
  p.rows_filled = (float)total_q_rows * y.heads_per_wg;
  if (!plan) {
    const auto schedule = ride ? attn_schedule_kernel<true> : attn_schedule_kernel<false>;
    schedule<<<1, kSchedThreads, 0, st>>>(n_req, ride ? x->req_off : d_q_off, p.q_off_out, d_matched_len, y.pos_log, p.max_items, y.units,
                                                      order_above(y, n_req, total_q_rows), p.rows_filled, p.n_items_out, (int32_t*)p.items, p.splits_out);
    SKV_HIP(hipGetLastError());
  }
  const int threads = y.two ? Form<true>::threads : kThreads;
  if (ride) {
    const auto kernel = y.two ? attn_rest_kernel<false, false, true>
                        : y.max_parts ? (plan ? attn_rest_kernel<true, true, false> : attn_rest_kernel<true, false, false>)
                                      : (plan ? attn_rest_kernel<false, true, false> : attn_rest_kernel<false, false, false>);
    const Rest rest = {x->gather, x->count, x->count.records ? n_req : 0, (int)grid};
    kernel<<<(int)grid + rest.n_count + std::min(skv_gather_blocks(x->gather), kCus), threads, 0, st>>>(p, rest);
  } else {
    const auto kernel = y.two ? attn_bf16_kernel<false, false, true>
                        : y.max_parts ? (plan ? attn_bf16_kernel<true, true, false> : attn_bf16_kernel<true, false, false>)
                                      : (plan ? attn_bf16_kernel<false, true, false> : attn_bf16_kernel<false, false, false>);
    kernel<<<(int)grid, threads, 0, st>>>(p);
  }
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
