// Index construction (host) and counter read-back / reset kernels.
//
// SafeKV Section 4.3.1 (Insert: blocks are appended along the radix-tree path, each entry
// recording private_tag and creator_id) and Section 4.3.2 (path compression: a chain is
// collapsed into one composite node that aggregates the KV addresses of the chain in a
// vector).  The tree is built without pointers: every distinct block-prefix gets an id
// through one hash table keyed by (parent id, 16 tokens); non-branching runs are then laid
// out contiguously and only branch points keep a child table.
#include <algorithm>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <numeric>
#include <new>
#include <vector>

#include "skv_internal.h"

static thread_local int g_last_hip_error = 0;
void skv_set_hip_error(int e) { g_last_hip_error = e; }

extern "C" int skv_last_hip_error(void) { return g_last_hip_error; }

extern "C" const char* skv_strerror(int code) {
  switch (code) {
    case SKV_OK: return "ok";
    case SKV_EINVAL: return "invalid argument";
    case SKV_ENOMEM: return "caller-provided device buffer too small";
    case SKV_ERANGE: return "value exceeds a built-in limit";
    case SKV_EHIP: return "HIP runtime error";
    default: return "unknown error";
  }
}

namespace {

constexpr int64_t kMaxBlocks = 0x7fffffff / 32;

struct Layout {  // byte offsets inside the slab
  size_t tok, page, meta, canon, flat_of, ctr, epoch, status, nodes, slots, total;
};

// Every array is sized for `cap` blocks: the entries the build creates plus room for later insertions.
// A node holds at least one block, so cap + 1 node records always suffice; child tables are kept at most
// half full and an outgrown table is left behind in the arena, which 8 slots per block cover.
size_t slots_for(size_t cap) { return 8 * cap + 8; }

Layout make_layout(size_t n_blocks, size_t n_in_blocks, size_t n_nodes_incl_root, size_t n_slots) {
  Layout l;
  size_t o = 0;
  l.tok = o;   o = skv_align256(o + n_blocks * 16 * sizeof(int32_t));
  l.page = o;  o = skv_align256(o + n_blocks * sizeof(int32_t));
  l.meta = o;  o = skv_align256(o + n_blocks * sizeof(int32_t));
  l.canon = o; o = skv_align256(o + n_blocks * sizeof(int32_t));
  l.flat_of = o; o = skv_align256(o + (n_in_blocks ? n_in_blocks : 1) * sizeof(int32_t));
  l.nodes = o; o = skv_align256(o + n_nodes_incl_root * sizeof(SkvNode));
  l.slots = o; o = skv_align256(o + (n_slots ? n_slots : 1) * sizeof(SkvSlot));
  l.ctr = o;   o = skv_align256(o + n_blocks * SKV_CTR_FIELDS * sizeof(uint32_t));
  l.epoch = o; o = skv_align256(o + (n_blocks ? n_blocks : 1) * sizeof(uint32_t));
  l.status = o; o = skv_align256(o + 64 * sizeof(uint32_t));   // word 0: limits the branching lookup ran into
  l.total = o;
  return l;
}

}  // namespace

// Host copy of the structure (not of the visibility bits or counters, which kernels change): what an
// insertion has to read and extend.
struct SkvHostMirror {
  Layout L;
  char* base = nullptr;               // the slab
  int64_t cap_blocks = 0;
  size_t slots_used = 0;
  std::vector<SkvNode> nodes;         // [n_nodes + 1]
  std::vector<int32_t> kids;          // children per node
  std::vector<int32_t> filled;        // table slots that are not empty (children + removed entries)
  std::vector<int32_t> parent;        // parent node of every node (root: -1)
  std::vector<SkvSlot> slots;         // the arena up to slots_used
  std::vector<int32_t> tok;           // [n_blocks][16], flat order
  std::vector<int32_t> canon, page;   // [n_blocks] input block id (-1 once evicted), page id
  std::vector<int32_t> flat_of;       // [n_in_blocks]
  std::vector<int32_t> node_of;       // [n_blocks] node that holds each block record (path ends name records)
  std::vector<uint8_t> page_used;     // [n_pages]
  int64_t live_blocks = 0;
  // Visibility words as the host last knew them.  Kernels change them (promotion, the safeguard's demotion), so
  // every call that enqueues such a kernel marks the copy stale and the next reader fetches it again.
  std::vector<int32_t> vis;           // [n_blocks]
  bool vis_stale = false;
  // Pinned memory small transfers go through: kStageBytes of it from the first write on, null before, and as long as none is
  // to be had.  Every call that uses it waits for its own kernels before it returns.
  char* stage = nullptr;
  // Kept for their memory only, nothing in them outlives a call: what a compaction lays out and changes places with, and marks per
  // page or input block.  Fresh from the allocator on every call they are faulted in again, 0.3 us per 4 KB.
  struct {
    std::vector<SkvNode> nodes;
    std::vector<SkvSlot> slots;
    std::vector<int32_t> kids, filled, parent;
  } saved;
  std::vector<uint32_t> words;
  std::vector<uint8_t> marks;
  void reserve_records(std::vector<int32_t>& tok, std::initializer_list<std::vector<int32_t>*> others) const {   // for a full slab
    tok.reserve((size_t)cap_blocks * 16);
    for (std::vector<int32_t>* v : others) v->reserve((size_t)cap_blocks);
  }
  ~SkvHostMirror();
  bool have_stage();
};

// Stages of trees that are gone.  skv_tree_destroy makes no runtime call (a collector may run it at any time, inside a stream
// capture too, where freeing pinned memory is an error): it leaves the stage here, linked through its first bytes.  The next
// tree to write takes one over, which also spares it the first touch of fresh pinned pages (0.4 ms per MB), and frees what is
// here beyond kParkedStages.
namespace {
constexpr size_t kStageBytes = 1 << 20;   // larger transfers are copies from and to ordinary memory (0.05 to 0.07 ms per MB)
constexpr int kParkedStages = 4;
struct Parked {
  Parked* next;
};
std::mutex parked_lock;
Parked* parked = nullptr;
}  // namespace

SkvHostMirror::~SkvHostMirror() {
  if (!stage) return;
  const std::lock_guard<std::mutex> hold(parked_lock);
  parked = new (stage) Parked{parked};
}

bool SkvHostMirror::have_stage() {
  if (stage) return true;
  Parked* rest = nullptr;
  {
    const std::lock_guard<std::mutex> hold(parked_lock);
    Parked** at = &parked;
    if (parked) {
      stage = (char*)parked;
      parked = parked->next;
    }
    for (int k = 0; *at && k < kParkedStages; ++k) at = &(*at)->next;
    std::swap(rest, *at);
  }
  while (rest) {
    Parked* const p = rest;
    rest = p->next;
    (void)hipHostFree(p);
  }
  if (!stage && hipHostMalloc((void**)&stage, kStageBytes, hipHostMallocPortable) != hipSuccess) {
    stage = nullptr;
    (void)hipGetLastError();   // no failure of the call: it copies instead
  }
  return stage != nullptr;
}

namespace {

int check_desc(const skv_tree_desc* d, int64_t* n_in_blocks) {
  if (!d || !d->seq_off) return SKV_EINVAL;
  if (d->block_tokens != SKV_BLOCK_TOKENS) return SKV_EINVAL;
  if (d->n_tenants < 1 || d->n_tenants > SKV_MAX_TENANTS) return SKV_ERANGE;
  if (d->n_pages < 1 || d->n_seq < 0) return SKV_EINVAL;
  if (d->seq_off[0] != 0) return SKV_EINVAL;
  for (int64_t s = 0; s < d->n_seq; ++s) {
    if (d->seq_off[s + 1] < d->seq_off[s] || d->seq_off[s + 1] % SKV_BLOCK_TOKENS) return SKV_EINVAL;
  }
  int64_t nib = d->seq_off[d->n_seq] / SKV_BLOCK_TOKENS;
  if (nib > kMaxBlocks) return SKV_ERANGE;
  if (nib > 0 && (!d->tokens || !d->blk_sensitive || !d->blk_owner || !d->blk_page)) return SKV_EINVAL;
  *n_in_blocks = nib;
  return SKV_OK;
}

Layout layout_for(size_t cap) { return make_layout(cap, cap, cap + 1, slots_for(cap)); }

uint32_t next_pow2(uint32_t x) {
  uint32_t p = 1;
  while (p < x) p <<= 1;
  return p;
}

__global__ void fill_u32_kernel(uint32_t* p, size_t n, uint32_t v) {
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
    p[i] = v;
}

// The read-backs run over the input blocks, in whose order the results lie: one pass that writes every element, default or
// not (a pass over the records behind one fill per result: 9.3 us for
// the three results of 263 k blocks, now 3.4).  A block that created no entry, or whose
// entry is gone, has no record.
__global__ void counters_read_kernel(SkvTreeDev t, int64_t n_in_blocks, uint32_t* hit, uint32_t* ucnt) {
  for (int64_t id = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; id < n_in_blocks; id += (int64_t)gridDim.x * blockDim.x) {
    const int b = t.flat_of[id];
    uint32_t h = 0, u = 0;
    if (b >= 0) {
      const uint32_t* c = t.ctr + b;
      h = c[0];
#pragma unroll
      for (int k = 1; k <= 4; ++k) u += __popc(c[k * t.ctr_plane]);
    }
    hit[id] = h;
    ucnt[id] = u;
  }
}

__global__ void counters_clear_window_kernel(SkvTreeDev t) {
  for (int b = blockIdx.x * blockDim.x + threadIdx.x; b < t.n_blocks; b += gridDim.x * blockDim.x) {
#pragma unroll
    for (int k = 0; k <= 4; ++k) t.ctr[k * t.ctr_plane + b] = 0;
  }
}

// Safeguard step (SafeKV Section 4.2.2, Section 6): one thread per block; a streaming pass over the
// counter planes (32 B read + 32 B written per block) and the metadata word.
__global__ void window_roll_kernel(SkvTreeDev t, skv_rdr_policy pol, int32_t* n_demoted) {
  for (int b0 = blockIdx.x * blockDim.x; b0 < t.n_blocks; b0 += gridDim.x * blockDim.x) {
    const int b = b0 + threadIdx.x;
    bool demote = false;
    if (b < t.n_blocks && t.canon[b] >= 0) {  // evicted records are skipped
      uint32_t* const c = t.ctr + b;
      const uint32_t h = c[0], u_pre = c[6 * t.ctr_plane], held = c[7 * t.ctr_plane];
      uint32_t u = 0;
#pragma unroll
      for (int k = 1; k <= 4; ++k) u += __popc(c[k * t.ctr_plane]);
      bool pred = false;
      if (h > 0 && h >= pol.min_hits) {
        const unsigned long long lhs = (unsigned long long)u * pol.tau_den, rhs = (unsigned long long)pol.tau_num * h;
        pred = pol.direction == 0 ? lhs < rhs : (lhs > rhs && u_pre <= pol.u_pre_max);
      }
      uint32_t streak = pred ? held + 1 : 0;
      const int m = t.meta[b];
      if (m >= 0 && streak >= pol.n_consec) {  // shareable (bit 31 clear) and the predicate held long enough
        t.meta[b] = m | (int)0x80000000;
        streak = 0;
        demote = true;
      }
#pragma unroll
      for (int k = 0; k <= 4; ++k) c[k * t.ctr_plane] = 0;
      c[5 * t.ctr_plane] = h;
      c[6 * t.ctr_plane] = u;
      c[7 * t.ctr_plane] = streak;
    }
    if (n_demoted) {
      const unsigned long long mask = __ballot(demote);
      if (mask && (threadIdx.x & 63) == 0) atomicAdd(n_demoted, (int)__popcll(mask));
    }
  }
}

__global__ void block_state_read_kernel(SkvTreeDev t, int64_t n_in_blocks, uint8_t* priv, uint32_t* hit_pre, uint32_t* u_pre) {
  for (int64_t id = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; id < n_in_blocks; id += (int64_t)gridDim.x * blockDim.x) {
    const int b = t.flat_of[id];
    const bool live = b >= 0;
    if (priv) priv[id] = live ? (t.meta[b] < 0 ? 1 : 0) : 255;
    if (hit_pre) hit_pre[id] = live ? t.ctr[5 * t.ctr_plane + b] : 0u;
    if (u_pre) u_pre[id] = live ? t.ctr[6 * t.ctr_plane + b] : 0u;
  }
}

__global__ void epochs_read_kernel(SkvTreeDev t, int64_t n_in_blocks, uint32_t* epoch) {
  for (int64_t id = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; id < n_in_blocks; id += (int64_t)gridDim.x * blockDim.x) {
    const int b = t.flat_of[id];
    epoch[id] = b >= 0 ? t.epoch[b] : 0u;
  }
}

__global__ void promote_kernel(SkvTreeDev t, int64_t n_in_blocks, const int32_t* ids, int n) {
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
    const int id = ids[i];
    if (id < 0 || id >= n_in_blocks) continue;
    const int f = t.flat_of[id];
    if (f >= 0) atomicAnd((unsigned int*)&t.meta[f], 0x7fffffffu);  // the visibility bit flips atomically
  }
}

// words [from, from + len) of every plane
__global__ void fill_planes_kernel(uint32_t* p, size_t plane, size_t from, size_t len, int planes) {
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < len * planes; i += (size_t)gridDim.x * blockDim.x)
    p[i / len * plane + from + i % len] = 0u;
}

// Words moved between the slab and the pinned memory, several spans in one launch (blockIdx.y).  One launch and one wait take
// the place of a copy per array, each through a staging buffer of the runtime's (64 requests, 7.7 k new blocks in an index of
// 67 k: insertion 192 -> 145 us, eviction 225 -> 150).
constexpr int kMaxSpans = 16;
struct Spans {
  uint32_t* dev[kMaxSpans];
  uint32_t* host[kMaxSpans];
  size_t words[kMaxSpans];
};
template <bool kUp>
__global__ void move_spans_kernel(Spans s) {
  const int k = blockIdx.y;
  uint32_t* const dst = kUp ? s.dev[k] : s.host[k];
  const uint32_t* const src = kUp ? s.host[k] : s.dev[k];
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < s.words[k]; i += (size_t)gridDim.x * blockDim.x) dst[i] = src[i];
}
// the records and input ids of evicted blocks
__global__ void evict_kernel(int32_t* canon, int32_t* flat_of, const int32_t* rec_id, int64_t n) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    canon[rec_id[2 * i]] = -1;
    flat_of[rec_id[2 * i + 1]] = -1;
  }
}

int grid_for(size_t n, int block) {
  size_t g = (n + block - 1) / block;
  if (g < 1) g = 1;
  if (g > 4096) g = 4096;
  return (int)g;
}

}  // namespace

extern "C" int skv_tree_build_size(const skv_tree_desc* desc, size_t* device_bytes) {
  int64_t nib = 0;
  int rc = check_desc(desc, &nib);
  if (rc) return rc;
  if (!device_bytes) return SKV_EINVAL;
  *device_bytes = layout_for((size_t)nib).total;
  return SKV_OK;
}

extern "C" int skv_tree_size_for_capacity(int64_t block_capacity, size_t* device_bytes) {
  if (block_capacity < 0 || !device_bytes) return SKV_EINVAL;
  if (block_capacity > kMaxBlocks) return SKV_ERANGE;
  *device_bytes = layout_for((size_t)block_capacity).total;
  return SKV_OK;
}

extern "C" int skv_tree_build(const skv_tree_desc* d, void* d_slab, size_t bytes, void* stream,
                              skv_tree** out) {
  int64_t nib64 = 0;
  int rc = check_desc(d, &nib64);
  if (rc) return rc;
  if (!out || !d_slab || ((uintptr_t)d_slab & 255)) return SKV_EINVAL;
  const int32_t nib = (int32_t)nib64;
  for (int32_t b = 0; b < nib; ++b) {
    if (d->blk_owner[b] < 0 || d->blk_owner[b] >= d->n_tenants) return SKV_EINVAL;
    if (d->blk_page[b] < 0 || d->blk_page[b] >= d->n_pages) return SKV_EINVAL;
  }

  // 1. one id per distinct block-prefix: hash table over (parent id, 16 tokens), first wins
  std::vector<int32_t> parent, src, n_child, only_child;
  std::vector<uint64_t> bhash;  // hash of the block's own 16 tokens
  parent.reserve(nib); src.reserve(nib); n_child.reserve(nib); only_child.reserve(nib); bhash.reserve(nib);
  const uint32_t cap = next_pow2((uint32_t)(2 * (size_t)nib + 2));
  std::vector<int32_t> table(cap, -1);
  for (int64_t s = 0; s < d->n_seq; ++s) {
    int32_t par = -1;
    for (int64_t b = d->seq_off[s] / 16; b < d->seq_off[s + 1] / 16; ++b) {
      const int32_t* tk = d->tokens + b * 16;
      const uint64_t hb = skv_hash_block_host(tk);
      uint32_t slot = (uint32_t)skv_hash_fin(hb + 0x632BE59BD9B4E019ull * (uint64_t)(uint32_t)(par + 1)) & (cap - 1);
      int32_t id;
      for (;;) {
        id = table[slot];
        if (id < 0) break;
        if (parent[id] == par && bhash[id] == hb && !memcmp(d->tokens + (size_t)src[id] * 16, tk, 64)) break;
        slot = (slot + 1) & (cap - 1);
      }
      if (id < 0) {
        id = (int32_t)parent.size();
        table[slot] = id;
        parent.push_back(par); src.push_back((int32_t)b); n_child.push_back(0);
        only_child.push_back(-1); bhash.push_back(hb);
        if (par >= 0) { n_child[par]++; only_child[par] = id; }
      }
      par = id;
    }
  }
  const int32_t n_blocks = (int32_t)parent.size();
  {  // one KV page may back only one cached block
    std::vector<uint8_t> used((size_t)d->n_pages, 0);
    for (int32_t b = 0; b < n_blocks; ++b) {
      int32_t p = d->blk_page[src[b]];
      if (used[p]) return SKV_EINVAL;
      used[p] = 1;
    }
  }

  // 2. nodes = maximal non-branching runs; flat order = node after node
  std::vector<int32_t> flat(n_blocks), node_of(n_blocks);
  std::vector<SkvNode> nodes(1, SkvNode{0, 0, 0, 0});
  std::vector<int32_t> head_of_node(1, -1);
  int32_t next_flat = 0;
  for (int32_t b = 0; b < n_blocks; ++b) {
    const bool head = parent[b] < 0 || n_child[parent[b]] != 1;
    if (!head) continue;
    SkvNode nd{next_flat, 0, 0, 0};
    const int32_t id = (int32_t)nodes.size();
    for (int32_t c = b;; c = only_child[c]) {
      flat[c] = next_flat++;
      node_of[c] = id;
      nd.n_blocks++;
      if (n_child[c] != 1) break;
    }
    nodes.push_back(nd);
    head_of_node.push_back(b);
  }
  const int32_t n_nodes = (int32_t)nodes.size() - 1;

  // 3. child tables at branch points
  std::vector<int32_t> kids(n_nodes + 1, 0);
  for (int32_t n = 1; n <= n_nodes; ++n) {
    int32_t p = parent[head_of_node[n]];
    kids[p < 0 ? 0 : node_of[p]]++;
  }
  size_t n_slots = 0;
  for (int32_t n = 0; n <= n_nodes; ++n) {
    nodes[n].tab_off = (int32_t)n_slots;
    nodes[n].tab_cap = kids[n] ? (int32_t)next_pow2(2u * (uint32_t)kids[n]) : 0;
    n_slots += (size_t)nodes[n].tab_cap;
  }
  if (n_slots > 0x7fffffff) return SKV_ERANGE;
  std::vector<SkvSlot> slots(n_slots ? n_slots : 1, SkvSlot{0, 0, -1, 0});
  for (int32_t n = 1; n <= n_nodes; ++n) {
    const int32_t hb = head_of_node[n];
    const SkvNode& pn = nodes[parent[hb] < 0 ? 0 : node_of[parent[hb]]];
    const uint64_t h = bhash[hb];
    uint32_t s = (uint32_t)h & (uint32_t)(pn.tab_cap - 1);
    while (slots[pn.tab_off + s].child >= 0) s = (s + 1) & (uint32_t)(pn.tab_cap - 1);
    slots[pn.tab_off + s] = SkvSlot{(uint32_t)h, (uint32_t)(h >> 32), n, 0};
  }

  // 4. stage and upload.  The slab's size fixes the capacity: the largest block count whose layout fits.
  if (layout_for((size_t)nib).total > bytes) return SKV_ENOMEM;
  int64_t cap_blocks = nib;
  for (int64_t lo = nib, hi = kMaxBlocks; lo <= hi;) {
    const int64_t mid = lo + (hi - lo) / 2;
    if (layout_for((size_t)mid).total <= bytes) { cap_blocks = mid; lo = mid + 1; } else { hi = mid - 1; }
  }
  const Layout L = layout_for((size_t)cap_blocks);
  if (n_slots > slots_for((size_t)cap_blocks)) return SKV_ENOMEM;
  std::vector<char> host(L.slots + (n_slots ? n_slots : 1) * sizeof(SkvSlot));  // everything up to the used slots
  int32_t* h_tok = (int32_t*)(host.data() + L.tok);
  int32_t* h_page = (int32_t*)(host.data() + L.page);
  int32_t* h_meta = (int32_t*)(host.data() + L.meta);
  int32_t* h_canon = (int32_t*)(host.data() + L.canon);
  int32_t* h_flat_of = (int32_t*)(host.data() + L.flat_of);
  for (int32_t b = 0; b < nib; ++b) h_flat_of[b] = -1;
  for (int32_t b = 0; b < n_blocks; ++b) {
    const int32_t f = flat[b], in = src[b];
    memcpy(h_tok + (size_t)f * 16, d->tokens + (size_t)in * 16, 64);
    h_page[f] = d->blk_page[in];
    h_meta[f] = (d->blk_sensitive[in] ? (int32_t)0x80000000 : 0) | d->blk_owner[in];
    h_canon[f] = in;
    h_flat_of[in] = f;
  }
  memcpy(host.data() + L.nodes, nodes.data(), nodes.size() * sizeof(SkvNode));
  memcpy(host.data() + L.slots, slots.data(), slots.size() * sizeof(SkvSlot));

  skv_tree* t = new (std::nothrow) skv_tree();
  if (!t) return SKV_EINVAL;
  char* base = (char*)d_slab;
  SkvHostMirror* m = new (std::nothrow) SkvHostMirror();
  if (!m) { delete t; return SKV_EINVAL; }
  t->host = m;
  t->has_copies = 0;
  m->L = L;
  m->base = base;
  m->cap_blocks = cap_blocks;
  m->slots_used = n_slots;
  m->nodes = nodes;
  m->kids = kids;
  m->filled = kids;
  m->parent.assign(nodes.size(), -1);
  for (int32_t n = 1; n <= n_nodes; ++n) {
    const int32_t pb = parent[head_of_node[n]];
    m->parent[n] = pb < 0 ? 0 : node_of[pb];
  }
  m->reserve_records(m->tok, {&m->canon, &m->page, &m->vis, &m->node_of, &m->flat_of});
  m->canon.assign(h_canon, h_canon + n_blocks);
  m->page.assign(h_page, h_page + n_blocks);
  m->vis.assign(h_meta, h_meta + n_blocks);
  m->node_of.assign((size_t)n_blocks, 0);
  for (int32_t n = 1; n <= n_nodes; ++n)
    for (int32_t k = 0; k < nodes[n].n_blocks; ++k) m->node_of[(size_t)nodes[n].first + k] = n;
  m->flat_of.assign(h_flat_of, h_flat_of + nib);
  m->live_blocks = n_blocks;
  m->slots.assign(slots.begin(), slots.begin() + n_slots);
  m->tok.assign(h_tok, h_tok + (size_t)n_blocks * 16);
  m->page_used.assign((size_t)d->n_pages, 0);
  for (int32_t b = 0; b < n_blocks; ++b) m->page_used[h_page[b]] = 1;
  t->dev.tok = (const int32_t*)(base + L.tok);
  t->dev.page = (const int32_t*)(base + L.page);
  t->dev.meta = (int32_t*)(base + L.meta);
  t->dev.canon = (const int32_t*)(base + L.canon);
  t->dev.flat_of = (const int32_t*)(base + L.flat_of);
  t->dev.ctr = (uint32_t*)(base + L.ctr);
  t->dev.ctr_plane = (size_t)cap_blocks;
  t->dev.epoch = (uint32_t*)(base + L.epoch);
  t->dev.limits = (uint32_t*)(base + L.status);
  t->dev.cur_epoch = 0;
  t->dev.nodes = (const SkvNode*)(base + L.nodes);
  t->dev.slots = (const SkvSlot*)(base + L.slots);
  t->dev.n_blocks = n_blocks;
  t->dev.n_nodes = n_nodes;
  t->dev.n_tenants = d->n_tenants;
  t->dev.n_pages = d->n_pages;
  t->n_in_blocks = nib;
  hipStream_t st = (hipStream_t)stream;
  hipError_t e = hipGetDevice(&t->device);
  if (e == hipSuccess) e = hipMemcpyAsync(base, host.data(), host.size(), hipMemcpyHostToDevice, st);
  if (e == hipSuccess && cap_blocks) {  // counters of the whole capacity: inserted blocks start from zero
    size_t n = (size_t)cap_blocks * SKV_CTR_FIELDS;
    fill_u32_kernel<<<grid_for(n, 256), 256, 0, st>>>(t->dev.ctr, n, 0u);
    fill_u32_kernel<<<grid_for((size_t)cap_blocks, 256), 256, 0, st>>>(t->dev.epoch, (size_t)cap_blocks, 0u);
    e = hipGetLastError();
  }
  if (e == hipSuccess) {
    fill_u32_kernel<<<1, 64, 0, st>>>(t->dev.limits, 64, 0u);
    e = hipGetLastError();
  }
  if (e == hipSuccess) e = hipStreamSynchronize(st);
  if (e != hipSuccess) {
    skv_set_hip_error((int)e);
    delete m;
    delete t;
    return SKV_EHIP;
  }
  *out = t;
  return SKV_OK;
}

// What one call moves between the slab and host memory: through the stage, one span behind the other, where it fits, otherwise
// a copy per span.
namespace {
struct Mover {
  SkvHostMirror* m;
  int n = 0;
  size_t bytes = 0;   // in the stage
  size_t dev_off[kMaxSpans], len[kMaxSpans];
  void* host[kMaxSpans];
  static size_t padded(size_t b) { return (b + 15) & ~(size_t)15; }
  void add(size_t off, const void* p, size_t b) {   // p stays valid until the call's wait
    if (!b) return;
    if (n < kMaxSpans) {
      dev_off[n] = off;
      host[n] = const_cast<void*>(p);
      len[n] = b;
    }
    bytes += padded(b);
    ++n;
  }
  template <bool kUp>
  int launch(hipStream_t st) const {
    Spans s;
    size_t at = 0, longest = 0;
    for (int k = 0; k < n; ++k) {
      s.dev[k] = (uint32_t*)(m->base + dev_off[k]);
      s.host[k] = (uint32_t*)(m->stage + at);
      s.words[k] = len[k] / 4;
      longest = std::max(longest, s.words[k]);
      if (kUp) memcpy(m->stage + at, host[k], len[k]);
      at += padded(len[k]);
    }
    if (n == 0) return SKV_OK;
    move_spans_kernel<kUp><<<dim3((unsigned)std::min<size_t>((longest + 255) / 256, 512), n), 256, 0, st>>>(s);
    SKV_HIP(hipGetLastError());
    return SKV_OK;
  }
  // Enqueues the upload; `behind`: bytes the caller wants in the stage behind the spans.  *staged: it went through the stage.
  int up(hipStream_t st, size_t behind = 0, bool* staged = nullptr) {
    if (n > kMaxSpans) return SKV_EINVAL;
    const bool fits = bytes + behind <= kStageBytes && m->have_stage();
    if (staged) *staged = fits;
    if (fits) return launch<true>(st);
    for (int k = 0; k < n; ++k) SKV_HIP(hipMemcpyAsync(m->base + dev_off[k], host[k], len[k], hipMemcpyHostToDevice, st));
    return SKV_OK;
  }
  // Fetches the spans and waits.  `in_place`: they may stay in the stage (-> true there), behind one another.
  int down(hipStream_t st, bool* in_place = nullptr) {
    if (n > kMaxSpans) return SKV_EINVAL;
    const bool fits = bytes <= kStageBytes && m->have_stage();
    if (fits) {
      const int rc = launch<false>(st);
      if (rc) return rc;
    } else {
      for (int k = 0; k < n; ++k) SKV_HIP(hipMemcpyAsync(host[k], m->base + dev_off[k], len[k], hipMemcpyDeviceToHost, st));
    }
    SKV_HIP(hipStreamSynchronize(st));
    if (in_place) {
      *in_place = fits;
    } else if (fits) {
      size_t at = 0;
      for (int k = 0; k < n; ++k) {
        memcpy(host[k], m->stage + at, len[k]);
        at += padded(len[k]);
      }
    }
    return SKV_OK;
  }
};
}  // namespace

// ---- insertion after prefill (Section 4.3.1 Insert; Section 4.1 and Section 6: new blocks are private by default) ----
namespace {

struct Inserter {
  skv_tree* t;
  SkvHostMirror* m;
  int64_t n_blocks, n_in;            // running totals
  size_t node_lo, node_hi, slot_lo, slot_hi;  // dirty spans of records that existed before [lo, hi)
  // What undo() needs: sizes before the call, and the records of then as they were before each change, oldest first.
  struct Node { int32_t at; SkvNode rec; int32_t kids, filled; };
  struct Slot { size_t at; SkvSlot rec; };
  struct Run { int32_t node, first, n; };   // a node's records that went to a new one, and its children with them
  std::vector<Node> old_nodes;
  std::vector<Slot> old_slots;
  std::vector<Run> cut;
  const size_t nodes0 = m->nodes.size(), slots0 = m->slots_used, blocks0 = m->canon.size(), in0 = m->flat_of.size();

  void keep_node(int32_t i) {
    if ((size_t)i < nodes0) old_nodes.push_back(Node{i, m->nodes[i], m->kids[i], m->filled[i]});
  }
  // Takes back everything the insertions so far did to the mirror.
  void undo() {
    for (size_t i = blocks0; i < m->page.size(); ++i) m->page_used[m->page[i]] = 0;
    for (size_t i = old_slots.size(); i-- > 0;) m->slots[old_slots[i].at] = old_slots[i].rec;
    for (size_t i = old_nodes.size(); i-- > 0;) {
      const Node& o = old_nodes[i];
      m->nodes[o.at] = o.rec; m->kids[o.at] = o.kids; m->filled[o.at] = o.filled;
    }
    m->nodes.resize(nodes0); m->kids.resize(nodes0); m->filled.resize(nodes0); m->parent.resize(nodes0);
    m->slots.resize(slots0); m->slots_used = slots0;
    m->tok.resize(blocks0 * 16); m->canon.resize(blocks0); m->page.resize(blocks0); m->vis.resize(blocks0); m->node_of.resize(blocks0);
    m->flat_of.resize(in0);
    for (const Run& c : cut) {
      if ((size_t)c.node >= nodes0) continue;   // of this call's own
      std::fill_n(m->node_of.begin() + c.first, c.n, c.node);
      const SkvNode& n = m->nodes[c.node];
      for (int32_t q = 0; q < n.tab_cap; ++q) {
        const int32_t child = m->slots[(size_t)n.tab_off + q].child;
        if (child >= 0) m->parent[child] = c.node;
      }
    }
  }

  void touch_node(size_t i) { node_lo = std::min(node_lo, i); node_hi = std::max(node_hi, i + 1); }
  void touch_slot(size_t i) { slot_lo = std::min(slot_lo, i); slot_hi = std::max(slot_hi, i + 1); }

  int32_t find_child(int32_t node, const int32_t* blk, uint64_t h) const {
    const SkvNode& n = m->nodes[node];
    if (!n.tab_cap) return -1;
    for (uint32_t s = (uint32_t)h & (uint32_t)(n.tab_cap - 1);; s = (s + 1) & (uint32_t)(n.tab_cap - 1)) {
      const SkvSlot& sl = m->slots[(size_t)n.tab_off + s];
      if (sl.child == -1) return -1;
      if (sl.child >= 0 && sl.hash_lo == (uint32_t)h && sl.hash_hi == (uint32_t)(h >> 32) &&
          !memcmp(&m->tok[(size_t)m->nodes[sl.child].first * 16], blk, 64))
        return sl.child;
    }
  }
  void put(int32_t node, uint64_t h, int32_t child) {  // into the first empty or removed slot of the probe sequence
    const SkvNode& n = m->nodes[node];
    uint32_t s = (uint32_t)h & (uint32_t)(n.tab_cap - 1);
    while (m->slots[(size_t)n.tab_off + s].child >= 0) s = (s + 1) & (uint32_t)(n.tab_cap - 1);
    if (m->slots[(size_t)n.tab_off + s].child == -1) m->filled[node]++;
    if ((size_t)n.tab_off + s < slots0) old_slots.push_back(Slot{(size_t)n.tab_off + s, m->slots[(size_t)n.tab_off + s]});
    m->slots[(size_t)n.tab_off + s] = SkvSlot{(uint32_t)h, (uint32_t)(h >> 32), child, 0};
    touch_slot((size_t)n.tab_off + s);
  }
  // Adds a child; a table that would become more than half full moves to a fresh one of twice the size.
  bool add_child(int32_t node, uint64_t h, int32_t child) {
    SkvNode& n = m->nodes[node];
    keep_node(node);
    const int32_t kids = m->kids[node] + 1;
    if (2 * (m->filled[node] + 1) > n.tab_cap) {  // removed entries count: a probe must always reach an empty slot
      const int32_t cap = (int32_t)next_pow2((uint32_t)(2 * kids) < 4u ? 4u : (uint32_t)(2 * kids));
      if (m->slots_used + (size_t)cap > slots_for((size_t)m->cap_blocks)) return false;
      const SkvNode old = n;
      n.tab_off = (int32_t)m->slots_used;
      n.tab_cap = cap;
      m->slots_used += (size_t)cap;
      m->slots.resize(m->slots_used, SkvSlot{0, 0, -1, 0});
      touch_slot((size_t)n.tab_off);
      touch_slot(m->slots_used - 1);
      m->filled[node] = 0;
      for (int32_t i = 0; i < old.tab_cap; ++i) {
        const SkvSlot sl = m->slots[(size_t)old.tab_off + i];
        if (sl.child >= 0) put(node, ((uint64_t)sl.hash_hi << 32) | sl.hash_lo, sl.child);
      }
      touch_node((size_t)node);
    }
    put(node, h, child);
    m->kids[node] = kids;
    return true;
  }
  // ---- private copies (Section 4.1): where the requester's own longest visible path ends ----
  // Several children of a node may start with the same block (one copy per tenant that could not see the others),
  // so the path is not unique and has to be searched: a stack of open positions, each with the copies that match
  // the request's next block ordered by the input id of their first block (the oldest copy is tried first).  A copy
  // is followed for as many blocks as match and are visible; if that covers the whole node the position below it
  // is opened, otherwise the path ends inside the node.  The first end that reaches the greatest depth is kept.
  struct PathEnd { int32_t node = 0, used = 0; int64_t depth = -1; };
  struct OpenPos {
    int32_t node;
    int64_t depth;
    std::vector<std::pair<int32_t, int32_t>> copies;  // (input id of the copy's first block, child node)
    size_t next = 0;
    bool extended = false;                             // some copy took the path further than this node
  };
  void matching_copies(int32_t node, const int32_t* blk, std::vector<std::pair<int32_t, int32_t>>& out) const {
    const SkvNode& n = m->nodes[node];
    if (!n.tab_cap) return;
    const uint64_t h = skv_hash_block_host(blk);
    const uint32_t mask = (uint32_t)(n.tab_cap - 1);
    for (uint32_t s = (uint32_t)h & mask; m->slots[(size_t)n.tab_off + s].child != -1; s = (s + 1) & mask) {
      const SkvSlot& sl = m->slots[(size_t)n.tab_off + s];
      if (sl.child < 0 || sl.hash_lo != (uint32_t)h || sl.hash_hi != (uint32_t)(h >> 32)) continue;
      const int32_t f = m->nodes[sl.child].first;
      if (!memcmp(&m->tok[(size_t)f * 16], blk, 64)) out.push_back({m->canon[f], sl.child});
    }
    std::sort(out.begin(), out.end());
  }
  int32_t visible_run(const SkvNode& c, const int32_t* x, int64_t room, int32_t tenant) const {
    const int64_t lim = std::min<int64_t>(c.n_blocks, room);
    int64_t k = 0;
    for (; k < lim; ++k) {
      const int32_t word = m->vis[(size_t)c.first + k];
      if (word < 0 && (word & 0x7fffffff) != tenant) break;   // private to somebody else
      if (memcmp(&m->tok[((size_t)c.first + k) * 16], x + k * 16, 64)) break;
    }
    return (int32_t)k;
  }
  PathEnd longest_visible_path(const int32_t* x, int64_t nb, int32_t tenant) const {
    PathEnd best;
    std::vector<OpenPos> open;
    auto open_at = [&](int32_t node, int64_t depth) {
      open.push_back(OpenPos{node, depth, {}});
      if (depth < nb) matching_copies(node, x + depth * 16, open.back().copies);
    };
    auto offer = [&](int32_t node, int32_t used, int64_t depth) {
      if (depth > best.depth) best = PathEnd{node, used, depth};
    };
    open_at(0, 0);
    while (!open.empty() && best.depth < nb) {
      OpenPos& p = open.back();
      if (p.next == p.copies.size()) {          // every copy tried: a position nothing continued is an end itself
        if (!p.extended) offer(p.node, m->nodes[p.node].n_blocks, p.depth);
        open.pop_back();
        continue;
      }
      const int32_t child = p.copies[p.next++].second;
      const SkvNode c = m->nodes[child];
      const int32_t k = visible_run(c, x + p.depth * 16, nb - p.depth, tenant);
      if (k == 0) continue;
      p.extended = true;
      const int64_t below = p.depth + k;        // (p may dangle after the next push)
      if (k == c.n_blocks) open_at(child, below);
      else offer(child, k, below);
    }
    return best;
  }
  // Appends blocks [k, nb) of the request below the end of its own longest visible path.  Returns k, or -1
  // when the slab is full.
  int64_t insert_copy(const int32_t* x, int64_t nb, int32_t tenant, const int32_t* pages, int64_t k_vis, int64_t* n_new) {
    *n_new = 0;
    const PathEnd end = longest_visible_path(x, nb, tenant);
    const int64_t k = end.depth;
    if (k >= nb || k < k_vis) return k;
    const int32_t at = end.node;
    if (end.used < m->nodes[at].n_blocks) {  // the path stops inside a compressed edge: split it there
      if ((int64_t)m->nodes.size() + 2 > m->cap_blocks + 1) return -1;
      if (!split(at, end.used)) return -1;
    }
    const int64_t add = nb - k;
    if (n_blocks + add > m->cap_blocks || n_in + add > m->cap_blocks) return -1;
    if ((int64_t)m->nodes.size() + 1 > m->cap_blocks + 1) return -1;
    return append(at, x, k, nb, tenant, pages, k_vis, n_new) ? k : -1;
  }
  // The same with the end of the requester's path given (the record of its last matched block, -1 for none; found by
  // the lookup before this batch).  What the lookup could not see are the blocks earlier requests of this batch added
  // for the same tenant; they hang below path ends the lookup did see, so the path is continued through them and
  // nothing else: a child (or the rest of a node) counts only if its blocks were created in this batch (records from
  // nb0 on) by this tenant.  Returns the index of the first new block, or -1 when the slab is full.
  int64_t insert_below(const int32_t* x, int64_t nb, int32_t tenant, const int32_t* pages, int64_t k_vis,
                       int32_t end_rec, int64_t nb0, int64_t* n_new) {
    *n_new = 0;
    int32_t node = 0, used = 0;
    if (end_rec >= 0) {
      node = m->node_of[end_rec];
      used = end_rec - m->nodes[node].first + 1;
    }
    int64_t k = k_vis;
    auto mine = [&](int32_t rec) { return rec >= nb0 && m->vis[rec] == ((int32_t)0x80000000 | tenant); };
    while (k < nb) {
      const SkvNode nd = m->nodes[node];
      if (used < nd.n_blocks) {              // inside a node: only this batch's own blocks continue the path
        const int32_t rec = nd.first + used;
        if (!mine(rec) || memcmp(&m->tok[(size_t)rec * 16], x + k * 16, 64)) break;
        ++used;
        ++k;
        continue;
      }
      int32_t next = -1;
      if (nd.tab_cap) {
        const uint64_t h = skv_hash_block_host(x + k * 16);
        const uint32_t mask = (uint32_t)(nd.tab_cap - 1);
        for (uint32_t q = (uint32_t)h & mask; m->slots[(size_t)nd.tab_off + q].child != -1; q = (q + 1) & mask) {
          const SkvSlot& sl = m->slots[(size_t)nd.tab_off + q];
          if (sl.child < 0 || sl.hash_lo != (uint32_t)h || sl.hash_hi != (uint32_t)(h >> 32)) continue;
          const int32_t rec = m->nodes[sl.child].first;
          if (mine(rec) && !memcmp(&m->tok[(size_t)rec * 16], x + k * 16, 64)) { next = sl.child; break; }
        }
      }
      if (next < 0) break;
      node = next;
      used = 1;
      ++k;
    }
    if (k >= nb) return k;
    if (used < m->nodes[node].n_blocks) {    // the path stops inside a compressed edge: split it there
      if ((int64_t)m->nodes.size() + 2 > m->cap_blocks + 1) return -1;
      if (!split(node, used)) return -1;
    }
    const int64_t add = nb - k;
    if (n_blocks + add > m->cap_blocks || n_in + add > m->cap_blocks) return -1;
    if ((int64_t)m->nodes.size() + 1 > m->cap_blocks + 1) return -1;
    return append(node, x, k, nb, tenant, pages, k_vis, n_new) ? k : -1;
  }
  // Cuts node c after its first j blocks: a new node takes the rest together with the child table.
  bool split(int32_t c, int64_t j) {
    const SkvNode run = m->nodes[c];
    keep_node(c);
    cut.push_back(Run{c, run.first + (int32_t)j, run.n_blocks - (int32_t)j});
    const int32_t tail = (int32_t)m->nodes.size();
    m->nodes.push_back(SkvNode{run.first + (int32_t)j, run.n_blocks - (int32_t)j, run.tab_off, run.tab_cap});
    m->kids.push_back(m->kids[c]);
    m->filled.push_back(m->filled[c]);
    m->parent.push_back(c);
    for (int32_t q = 0; q < run.tab_cap; ++q) {  // the children move below the new node
      const int32_t gc = m->slots[(size_t)run.tab_off + q].child;
      if (gc >= 0) m->parent[gc] = tail;
    }
    for (int32_t k = (int32_t)j; k < run.n_blocks; ++k) m->node_of[(size_t)run.first + k] = tail;
    m->nodes[c].n_blocks = (int32_t)j;
    m->nodes[c].tab_off = 0;
    m->nodes[c].tab_cap = 0;
    m->kids[c] = 0;
    m->filled[c] = 0;
    touch_node((size_t)c);
    touch_node((size_t)tail);
    return add_child(c, skv_hash_block_host(&m->tok[((size_t)run.first + j) * 16]), tail);
  }
  // New node with blocks [i, nb) of the request as a child of `node`.
  bool append(int32_t node, const int32_t* x, int64_t i, int64_t nb, int32_t tenant, const int32_t* pages,
              int64_t k_vis, int64_t* n_new) {
    const int64_t add = nb - i;
    const int32_t fresh = (int32_t)m->nodes.size();
    m->nodes.push_back(SkvNode{(int32_t)n_blocks, (int32_t)add, 0, 0});
    m->kids.push_back(0);
    m->filled.push_back(0);
    m->parent.push_back(node);
    touch_node((size_t)fresh);
    if (!add_child(node, skv_hash_block_host(x + i * 16), fresh)) return false;
    // (an array at a time, which the upload then reads where it lies: 64 requests with 7.7 k new blocks 116 -> 90 us a call, 40 of it
    // upload and wait; a block at a time went through eleven vectors)
    const int32_t* const own = pages + (i - k_vis);
    m->tok.insert(m->tok.end(), x + i * 16, x + nb * 16);
    m->vis.insert(m->vis.end(), (size_t)add, (int32_t)0x80000000 | tenant);
    m->node_of.insert(m->node_of.end(), (size_t)add, fresh);
    m->page.insert(m->page.end(), own, own + add);
    const size_t c0 = m->canon.size(), f0 = m->flat_of.size();
    m->canon.resize(c0 + (size_t)add);
    m->flat_of.resize(f0 + (size_t)add);
    std::iota(m->canon.begin() + c0, m->canon.end(), (int32_t)n_in);
    std::iota(m->flat_of.begin() + f0, m->flat_of.end(), (int32_t)n_blocks);
    for (int64_t j = 0; j < add; ++j) m->page_used[own[j]] = 1;
    n_blocks += add;
    n_in += add;
    *n_new = add;
    return true;
  }
  // One request: blocks [k_exist, nb) are appended as one node below the point where the path ends.
  // Returns k_exist, or -1 when the slab is full.
  int64_t insert(const int32_t* x, int64_t nb, int32_t tenant, const int32_t* pages, int64_t k_vis, int64_t* n_new) {
    *n_new = 0;
    int32_t node = 0;
    int64_t i = 0;
    while (i < nb) {
      const uint64_t h = skv_hash_block_host(x + i * 16);
      const int32_t c = find_child(node, x + i * 16, h);
      if (c < 0) break;
      const SkvNode run = m->nodes[c];
      int64_t j = 1;
      while (j < run.n_blocks && i + j < nb && !memcmp(&m->tok[((size_t)run.first + j) * 16], x + (i + j) * 16, 64)) ++j;
      if (j < run.n_blocks) {
        if (i + j == nb) return nb;  // the request ends inside the run: nothing new
        if (i + j < k_vis) return i + j;  // caller's matched length is not one this tree gives
        // split: the run keeps its first j blocks, a new node takes the rest together with the child table
        if ((int64_t)m->nodes.size() + 2 > m->cap_blocks + 1) return -1;
        if (!split(c, j)) return -1;
        node = c;
        i += j;
        break;
      }
      node = c;
      i += j;
    }
    if (i >= nb || i < k_vis) return i;
    const int64_t add = nb - i;
    if (n_blocks + add > m->cap_blocks || n_in + add > m->cap_blocks) return -1;
    if (!append(node, x, i, nb, tenant, pages, k_vis, n_new)) return -1;
    return i;
  }
};

}  // namespace

extern "C" int skv_tree_insert(skv_tree* t, int32_t n_req, const int32_t* req_off, const int32_t* req_tokens,
                               const int32_t* req_tenant, const int32_t* matched_len, const int32_t* new_pages,
                               int32_t max_new_blocks, int32_t private_copies, const int32_t* path_end,
                               int32_t* first_inserted, int32_t* n_inserted, void* stream) {
  if (!t || !t->host || n_req < 0 || max_new_blocks < 0) return SKV_EINVAL;
  if (n_req == 0) return SKV_OK;
  if (!req_off || !req_tenant || !matched_len || !first_inserted || !n_inserted) return SKV_EINVAL;
  if (max_new_blocks > 0 && !new_pages) return SKV_EINVAL;
  SkvHostMirror* m = t->host;
  // validate everything before anything changes
  std::vector<int32_t> have(n_req, 0);
  {
    std::vector<uint8_t>& seen = m->marks;
    seen.assign(m->page_used.size(), 0);
    for (int32_t r = 0; r < n_req; ++r) {
      if (req_off[r + 1] < req_off[r] || req_off[r] < 0 || matched_len[r] < 0) return SKV_EINVAL;
      if (req_off[r + 1] > req_off[r] && !req_tokens) return SKV_EINVAL;
      if (req_tenant[r] < 0 || req_tenant[r] >= t->dev.n_tenants) return SKV_EINVAL;
      int32_t h = 0;
      for (; h < max_new_blocks; ++h) {
        const int32_t pg = new_pages[(size_t)r * max_new_blocks + h];
        if (pg < 0) break;
        if (pg >= t->dev.n_pages || m->page_used[pg] || seen[pg]) return SKV_EINVAL;
        seen[pg] = 1;
      }
      have[r] = h;
      if (private_copies && path_end) {   // the record must be this request's last matched block
        const int64_t k_vis = matched_len[r] / SKV_BLOCK_TOKENS;
        const int32_t e = path_end[r];
        if (k_vis == 0 ? e != -1
                       : (e < 0 || e >= t->dev.n_blocks || m->canon[e] < 0 ||
                          k_vis * SKV_BLOCK_TOKENS > req_off[r + 1] - req_off[r] ||
                          memcmp(&m->tok[(size_t)e * 16], req_tokens + req_off[r] + (k_vis - 1) * 16, 64)))
          return SKV_EINVAL;
      }
    }
  }
  // Work on the mirror; where the slab is full every change is taken back.  (From records kept of what changed: a snapshot is a copy of
  // the index's size, 116 instead of 97 us for 64 requests, 7.7 k new blocks in 67 k.)
  Inserter ins{t, m, t->dev.n_blocks, t->n_in_blocks, SIZE_MAX, 0, SIZE_MAX, 0};
  hipStream_t st = (hipStream_t)stream;
  // The requester's own path depends on the visibility bits.  The host's copy of them is exact unless a
  // promotion or a safeguard window has been enqueued since it was taken; only then is it fetched again.
  if (private_copies && !path_end && m->vis_stale && t->dev.n_blocks) {
    SKV_HIP(hipMemcpyAsync(m->vis.data(), t->dev.meta, (size_t)t->dev.n_blocks * 4, hipMemcpyDeviceToHost, st));
    SKV_HIP(hipStreamSynchronize(st));
    m->vis_stale = false;
  }
  bool full = false;
  for (int32_t r = 0; r < n_req && !full; ++r) {
    const int64_t k_vis = matched_len[r] / SKV_BLOCK_TOKENS;
    int64_t nb = (req_off[r + 1] - req_off[r]) / SKV_BLOCK_TOKENS;
    if (nb > k_vis + have[r]) nb = k_vis + have[r];
    int64_t n_new = 0;
    const int32_t* pages_r = new_pages + (size_t)r * max_new_blocks;
    const int32_t* x = req_tokens + req_off[r];
    const int64_t first = !private_copies ? ins.insert(x, nb, req_tenant[r], pages_r, k_vis, &n_new)
                          : path_end      ? ins.insert_below(x, nb, req_tenant[r], pages_r, k_vis, path_end[r], t->dev.n_blocks, &n_new)
                                          : ins.insert_copy(x, nb, req_tenant[r], pages_r, k_vis, &n_new);
    if (first < 0) { full = true; break; }
    first_inserted[r] = (int32_t)first;
    n_inserted[r] = (int32_t)n_new;
  }
  if (full) {
    ins.undo();
    return SKV_ENOMEM;
  }
  // upload: the appended block records, then the spans of node and slot records that changed
  const int64_t nb0 = t->dev.n_blocks, nin0 = t->n_in_blocks, add = ins.n_blocks - nb0;
  if (private_copies && add > 0) t->has_copies = 1;
  const std::vector<uint32_t> epochs((size_t)add, t->dev.cur_epoch);
  const size_t n_node = ins.node_hi > ins.node_lo ? ins.node_hi - ins.node_lo : 0, n_slot = ins.slot_hi > ins.slot_lo ? ins.slot_hi - ins.slot_lo : 0;
  Mover up{m};
  up.add(m->L.tok + (size_t)nb0 * 64, m->tok.data() + (size_t)nb0 * 16, (size_t)add * 64);
  up.add(m->L.page + (size_t)nb0 * 4, m->page.data() + nb0, (size_t)add * 4);
  up.add(m->L.meta + (size_t)nb0 * 4, m->vis.data() + nb0, (size_t)add * 4);
  up.add(m->L.canon + (size_t)nb0 * 4, m->canon.data() + nb0, (size_t)add * 4);
  up.add(m->L.flat_of + (size_t)nin0 * 4, m->flat_of.data() + nin0, (size_t)add * 4);
  up.add(m->L.epoch + (size_t)nb0 * 4, epochs.data(), (size_t)add * 4);
  if (n_node) up.add(m->L.nodes + ins.node_lo * sizeof(SkvNode), &m->nodes[ins.node_lo], n_node * sizeof(SkvNode));
  if (n_slot) up.add(m->L.slots + ins.slot_lo * sizeof(SkvSlot), &m->slots[ins.slot_lo], n_slot * sizeof(SkvSlot));
  const int rc = up.up(st);
  if (rc) return rc;
  SKV_HIP(hipStreamSynchronize(st));
  t->dev.n_blocks = (int32_t)ins.n_blocks;
  t->dev.n_nodes = (int32_t)m->nodes.size() - 1;
  t->n_in_blocks = ins.n_in;
  m->live_blocks += add;
  return SKV_OK;
}

// ---- eviction (Section 4.3.1 Evict: epoch-based LRU; Section 4.3.2 progressive eviction) ----
extern "C" int skv_set_epoch(skv_tree* t, uint32_t epoch) {
  if (!t) return SKV_EINVAL;
  t->dev.cur_epoch = epoch;
  return SKV_OK;
}

extern "C" int skv_block_epochs_read(skv_tree* t, uint32_t* d_epoch, void* stream) {
  if (!t || !d_epoch) return SKV_EINVAL;
  hipStream_t st = (hipStream_t)stream;
  if (t->n_in_blocks) epochs_read_kernel<<<grid_for((size_t)t->n_in_blocks, 256), 256, 0, st>>>(t->dev, t->n_in_blocks, d_epoch);
  SKV_HIP(hipGetLastError());
  return SKV_OK;
}

extern "C" int skv_evict(skv_tree* t, int64_t n_want, const int32_t* protect_ids, int64_t n_protect,
                         int32_t* evicted_ids, int32_t* evicted_pages, int64_t* n_evicted, void* stream) {
  if (!t || !t->host || n_want < 0 || n_protect < 0 || !n_evicted) return SKV_EINVAL;
  if (n_protect > 0 && !protect_ids) return SKV_EINVAL;
  if (n_want > 0 && (!evicted_ids || !evicted_pages)) return SKV_EINVAL;
  *n_evicted = 0;
  SkvHostMirror* m = t->host;
  const int64_t nb = t->dev.n_blocks;
  if (n_want == 0 || nb == 0) return SKV_OK;
  hipStream_t st = (hipStream_t)stream;
  std::vector<uint32_t> own;
  if ((size_t)nb * 4 > kStageBytes || !m->have_stage()) own.resize((size_t)nb);
  Mover down{m};
  down.add(m->L.epoch, own.data(), (size_t)nb * 4);
  bool in_stage = false;
  int rc = down.down(st, &in_stage);
  if (rc) return rc;
  const uint32_t* const epoch = in_stage ? (const uint32_t*)m->stage : own.data();
  std::vector<uint8_t>& prot = m->marks;
  prot.assign((size_t)t->n_in_blocks, 0);
  constexpr int64_t kRun = 64;   // ids mostly come in runs
  for (int64_t i = 0; i < n_protect;) {
    const int64_t n = std::min(kRun, n_protect - i);
    const int32_t first = protect_ids[i];
    int32_t off = 0;
    for (int64_t k = 0; k < n; ++k) off |= (int32_t)((uint32_t)protect_ids[i + k] - (uint32_t)first) ^ (int32_t)k;
    if (off == 0 && first >= 0 && first + n <= t->n_in_blocks) {
      memset(&prot[first], 1, (size_t)n);
    } else {
      for (int64_t k = 0; k < n; ++k)
        if (protect_ids[i + k] >= 0 && protect_ids[i + k] < t->n_in_blocks) prot[protect_ids[i + k]] = 1;
    }
    i += n;
  }
  // candidates: the last block of every childless node, oldest (epoch, block id) first
  struct Cand { uint32_t epoch; int32_t id, node; };
  auto later = [](const Cand& a, const Cand& b) { return a.epoch != b.epoch ? a.epoch > b.epoch : a.id > b.id; };
  std::vector<Cand> heap;
  auto tail_of = [&](int32_t n) {
    const SkvNode& nd = m->nodes[n];
    const int32_t f = nd.first + nd.n_blocks - 1;
    return Cand{epoch[f], m->canon[f], n};
  };
  auto push_tail = [&](int32_t n) {   // (of a node whose children have all gone)
    heap.push_back(tail_of(n));
    std::push_heap(heap.begin(), heap.end(), later);
  };
  for (int32_t n = 1; n < (int32_t)m->nodes.size(); ++n) {
    if (m->kids[n] || m->nodes[n].n_blocks <= 0) continue;
    const Cand tail = tail_of(n);
    if (!prot[tail.id]) heap.push_back(tail);   // (in use: the node keeps its tail, and with it everything above)
  }
  std::make_heap(heap.begin(), heap.end(), later);
  size_t node_lo = SIZE_MAX, node_hi = 0, slot_lo = SIZE_MAX, slot_hi = 0;
  std::vector<int32_t> gone(2 * (size_t)std::min(n_want, nb));   // record and input id of every evicted block
  int64_t done = 0;
  while (done < n_want && !heap.empty()) {
    std::pop_heap(heap.begin(), heap.end(), later);
    const Cand c = heap.back();
    heap.pop_back();
    SkvNode& nd = m->nodes[c.node];
    // A node's blocks mostly go one after another: from its last one up to one that is in use (the node keeps it, and with it everything
    // above) or younger than the oldest in the heap.  How many first, and then each array in a loop of its own
    // (a call that evicts 7.6 k of 75 k blocks 97 -> 84 us with the wait for epochs and upload, about 40 of it).
    const int32_t first = nd.first, tail = first + nd.n_blocks - 1;
    const int32_t least = (int32_t)std::max<int64_t>(first, tail + 1 - (n_want - done));
    int32_t f = tail;   // the last block that stays
    bool younger = false;
    for (; f >= least && !prot[m->canon[f]]; --f) {
      younger = f < tail && !heap.empty() && later(Cand{epoch[f], m->canon[f], c.node}, heap.front());
      if (younger) break;
    }
    const int32_t n = tail - f;
    int32_t *const ids = evicted_ids + done, *const pages = evicted_pages + done, *const pairs = gone.data() + 2 * done;
    for (int32_t i = 0; i < n; ++i) ids[i] = m->canon[tail - i];
    for (int32_t i = 0; i < n; ++i) pages[i] = m->page[tail - i];
    for (int32_t i = 0; i < n; ++i) {
      pairs[2 * i] = tail - i;
      pairs[2 * i + 1] = ids[i];
    }
    for (int32_t i = 0; i < n; ++i) m->page_used[pages[i]] = 0;
    for (int32_t i = 0; i < n; ++i) m->flat_of[ids[i]] = -1;
    std::fill_n(m->canon.begin() + f + 1, n, -1);
    done += n;
    if (younger) {
      heap.push_back(Cand{epoch[f], m->canon[f], c.node});
      std::push_heap(heap.begin(), heap.end(), later);
    }
    nd.n_blocks = f + 1 - first;
    node_lo = std::min(node_lo, (size_t)c.node); node_hi = std::max(node_hi, (size_t)c.node + 1);
    if (nd.n_blocks > 0) continue;
    // the node is gone: its entry in the parent's table becomes a removed slot
    const int32_t p = m->parent[c.node];
    const SkvNode& pn = m->nodes[p];
    for (int32_t q = 0; q < pn.tab_cap; ++q) {
      SkvSlot& sl = m->slots[(size_t)pn.tab_off + q];
      if (sl.child == c.node) {
        sl.child = -2;
        slot_lo = std::min(slot_lo, (size_t)pn.tab_off + q); slot_hi = std::max(slot_hi, (size_t)pn.tab_off + q + 1);
        break;
      }
    }
    m->kids[p]--;
    if (m->kids[p] == 0 && p != 0 && pn.n_blocks > 0) push_tail(p);
  }
  *n_evicted = done;
  m->live_blocks -= done;
  if (!done) return SKV_OK;
  const size_t n_node = node_hi - node_lo, n_slot = slot_hi > slot_lo ? slot_hi - slot_lo : 0;   // (a block is gone: so a node changed)
  Mover up{m};
  up.add(m->L.nodes + node_lo * sizeof(SkvNode), &m->nodes[node_lo], n_node * sizeof(SkvNode));
  if (n_slot) up.add(m->L.slots + slot_lo * sizeof(SkvSlot), &m->slots[slot_lo], n_slot * sizeof(SkvSlot));
  bool staged;
  gone.resize(2 * (size_t)done);
  rc = up.up(st, gone.size() * 4, &staged);
  if (rc) return rc;
  if (staged) {
    int32_t* const rec_id = (int32_t*)(m->stage + up.bytes);
    memcpy(rec_id, gone.data(), gone.size() * 4);
    evict_kernel<<<grid_for((size_t)done, 256), 256, 0, st>>>((int32_t*)(m->base + m->L.canon), (int32_t*)(m->base + m->L.flat_of), rec_id, done);
    SKV_HIP(hipGetLastError());
  } else {
    size_t blk_lo = SIZE_MAX, blk_hi = 0, id_lo = SIZE_MAX, id_hi = 0;
    for (int64_t i = 0; i < done; ++i) {
      const size_t f = (size_t)gone[2 * i], id = (size_t)gone[2 * i + 1];
      blk_lo = std::min(blk_lo, f); blk_hi = std::max(blk_hi, f + 1);
      id_lo = std::min(id_lo, id); id_hi = std::max(id_hi, id + 1);
    }
    SKV_HIP(hipMemcpyAsync(m->base + m->L.canon + blk_lo * 4, &m->canon[blk_lo], (blk_hi - blk_lo) * 4, hipMemcpyHostToDevice, st));
    SKV_HIP(hipMemcpyAsync(m->base + m->L.flat_of + id_lo * 4, &m->flat_of[id_lo], (id_hi - id_lo) * 4, hipMemcpyHostToDevice, st));
  }
  SKV_HIP(hipStreamSynchronize(st));
  return SKV_OK;
}

// ---- reclaiming record space (Section 4.3.2 Progressive Eviction: a chain's address vector shrinks as its entries
// are released and the chain itself goes once the vector is empty) ----
// Evictions shorten node runs and unlink emptied nodes, insertions abandon outgrown child tables and split runs; the
// records they leave behind stay in the slab.  Compaction closes the gaps: block records, nodes and input block ids keep their order
// (so "older copy" and eviction ties still compare the same way) and move up, child tables are laid out afresh for the children they
// have.  What lies before the first gap stays where it is, on the device too, so the cost is that of the nodes and of what moves; of that,
// the per-block state the kernels own (visibility bits, counters, epochs) is read back, moved with the records and written again.
// (67 k blocks in 1.5 k nodes, ten rounds of 7.7 k inserted and evicted behind them: 106 us, laid out afresh throughout 1090; where
// blocks go from everywhere the host's part is 0.85 ms for 17 k to 51 k that move.)  Nodes in the order of a walk instead of the order they
// were made in would be worth 1 % of a lookup where every prompt was split many times (24 rounds, 2648 nodes in 40 k blocks, 64 requests
// 36.8 / 36.0 us, 4096 36.0 / 35.8) and cost every compaction 60 us.
extern "C" int skv_tree_compact(skv_tree* t, int32_t* id_map, int64_t* n_in_blocks_after, void* stream) {
  if (!t || !t->host) return SKV_EINVAL;
  SkvHostMirror* m = t->host;
  hipStream_t st = (hipStream_t)stream;
  const size_t nb_old = (size_t)t->dev.n_blocks, nin_old = (size_t)t->n_in_blocks, live = (size_t)m->live_blocks;
  if (nin_old > 0 && !id_map) return SKV_EINVAL;
  const size_t plane = t->dev.ctr_plane;
  const Layout& L = m->L;
  size_t f0 = 0, d0 = 0;   // the first record, and input id, that is gone
  while (f0 < nb_old && m->canon[f0] >= 0) ++f0;
  while (d0 < nin_old && m->flat_of[d0] >= 0) ++d0;
  size_t d1 = nin_old;     // behind the last input id that is there
  while (d1 > d0 && m->flat_of[d1 - 1] < 0) --d1;
  std::vector<std::pair<int32_t, int32_t>> moved;   // nodes behind the gap, in the order of their records, and their new first record
  size_t n_live = f0, id_lo = d0;   // id_lo, canon_lo: the first input id whose record changes, the first record whose id does
  for (size_t f = f0; f < nb_old;) {
    if (m->canon[f] < 0) {
      ++f;
      continue;
    }
    const int32_t n = m->node_of[f];
    const SkvNode& nd = m->nodes[n];
    if ((size_t)nd.first != f || nd.n_blocks <= 0 || f + (size_t)nd.n_blocks > nb_old) return SKV_EINVAL;   // the mirror lost track of a block: refuse rather than drop it
    moved.push_back({n, (int32_t)n_live});
    n_live += (size_t)nd.n_blocks;
    for (const size_t end = f + (size_t)nd.n_blocks; f < end; ++f) id_lo = std::min(id_lo, (size_t)m->canon[f]);
  }
  if (n_live != live) return SKV_EINVAL;
  uint32_t canon_lo = (uint32_t)f0;
  for (size_t i = d0; i < d1; ++i) canon_lo = std::min(canon_lo, (uint32_t)m->flat_of[i]);   // (-1: none)
  // Laid out beside the mirror, which takes it over once the slab holds it: a call that fails leaves the mirror, the counts and id_map as
  // they were.  Tokens and pages, most of the bytes, are moved in the mirror and back again if it comes to that (with them copied
  // out and in as well a compaction that moves 35 k blocks takes the host 1.1 ms instead of 0.8).
  constexpr int kOwned = 2 + SKV_CTR_FIELDS;
  const size_t n_read = live > f0 ? nb_old - f0 : 0, n_write = live - f0, n_flat = d1 - id_lo, n_canon = live - canon_lo, n_id = d1 - d0;
  m->words.resize((n_read + n_write) * kOwned + n_flat + n_canon + n_id);
  int32_t *const flat_of = (int32_t*)m->words.data() + (n_read + n_write) * kOwned, *const canon = flat_of + n_flat, *const new_id = canon + n_canon;   // from id_lo, canon_lo, d0 on
  // what the kernels own of the records that move, as the device has it: visibility, epochs, counter planes
  uint32_t *state[kOwned], *n_state[kOwned];
  size_t off[kOwned];
  for (int q = 0; q < kOwned; ++q) {
    state[q] = m->words.data() + n_read * q;
    n_state[q] = m->words.data() + n_read * kOwned + n_write * q;
    off[q] = (q == 0 ? L.meta : q == 1 ? L.epoch : L.ctr + (q - 2) * plane * 4) + f0 * 4;
  }
  Mover down{m};
  for (int q = 0; q < kOwned; ++q) down.add(off[q], state[q], n_read * 4);
  int rc = n_read ? down.down(st) : SKV_OK;
  if (rc) return rc;
  // records
  std::copy_n(m->flat_of.begin() + id_lo, n_flat, flat_of);
  std::copy_n(m->canon.begin() + canon_lo, f0 - canon_lo, canon);
  for (const auto& [n, to] : moved) {
    const size_t f = (size_t)m->nodes[n].first, k = (size_t)m->nodes[n].n_blocks, g = (size_t)to - f0;
    for (int q = 0; q < kOwned; ++q) memcpy(n_state[q] + g, state[q] + (f - f0), k * 4);
    for (size_t i = 0; i < k; ++i) {
      canon[(size_t)to + i - canon_lo] = m->canon[f + i];
      flat_of[(size_t)m->canon[f + i] - id_lo] = to + (int32_t)i;
    }
  }
  // dense input ids, old order kept
  size_t n_ids = d0;
  for (size_t i = d0; i < d1; ++i) {
    const int32_t f = flat_of[i - id_lo];
    new_id[i - d0] = f < 0 ? -1 : (int32_t)n_ids;
    if (f < 0) continue;
    canon[(size_t)f - canon_lo] = (int32_t)n_ids;
    flat_of[n_ids++ - id_lo] = f;
  }
  // nodes, and their tables
  std::vector<SkvNode>& nodes = m->saved.nodes;
  std::vector<SkvSlot>& slots = m->saved.slots;
  std::vector<int32_t>&kids = m->saved.kids, &filled = m->saved.filled, &parent = m->saved.parent;
  nodes.clear(); slots.clear(); kids.clear(); filled.clear(); parent.clear();
  std::vector<int32_t> new_node(m->nodes.size(), -1);
  int32_t n_nodes = 0;
  for (size_t n = 0; n < m->nodes.size(); ++n)
    if (n == 0 || m->nodes[n].n_blocks > 0) new_node[n] = n_nodes++;
  for (size_t n = 0; n < m->nodes.size(); ++n) {
    if (new_node[n] < 0) continue;
    SkvNode nd = m->nodes[n];
    const SkvSlot* const old = m->slots.data() + nd.tab_off;
    int32_t n_kids = 0;
    for (int32_t q = 0; q < nd.tab_cap; ++q) n_kids += old[q].child >= 0;
    const int32_t old_cap = nd.tab_cap;
    nd.tab_off = nd.tab_cap = 0;
    if (n_kids) {
      const uint32_t cap = next_pow2((uint32_t)std::max(4, 2 * n_kids));
      nd.tab_off = (int32_t)slots.size();
      nd.tab_cap = (int32_t)cap;
      slots.resize(slots.size() + cap, SkvSlot{0, 0, -1, 0});
      for (int32_t q = 0; q < old_cap; ++q) {
        if (old[q].child < 0) continue;
        uint32_t at = old[q].hash_lo & (cap - 1);
        while (slots[(size_t)nd.tab_off + at].child >= 0) at = (at + 1) & (cap - 1);
        slots[(size_t)nd.tab_off + at] = SkvSlot{old[q].hash_lo, old[q].hash_hi, new_node[old[q].child], 0};
      }
    }
    nodes.push_back(nd);
    kids.push_back(n_kids);
    filled.push_back(n_kids);
    parent.push_back(m->parent[n] < 0 ? -1 : new_node[m->parent[n]]);
  }
  for (const auto& [n, to] : moved) nodes[new_node[n]].first = to;
  // (nothing is allocated in the mirror from here on)
  auto move_block = [&](size_t from, size_t to, size_t k) {
    memmove(&m->tok[to * 16], &m->tok[from * 16], k * 64);
    memmove(&m->page[to], &m->page[from], k * 4);
  };
  for (const auto& [n, to] : moved) move_block((size_t)m->nodes[n].first, (size_t)to, (size_t)m->nodes[n].n_blocks);
  // write back what changed; counters and epochs of the free records start from zero again
  auto write_back = [&]() -> int {
    Mover up{m};
    up.add(L.tok + f0 * 64, m->tok.data() + f0 * 16, n_write * 64);
    up.add(L.page + f0 * 4, m->page.data() + f0, n_write * 4);
    up.add(L.canon + canon_lo * 4, canon, n_canon * 4);
    up.add(L.flat_of + id_lo * 4, flat_of, (n_ids - id_lo) * 4);
    up.add(L.nodes, nodes.data(), nodes.size() * sizeof(SkvNode));
    up.add(L.slots, slots.data(), slots.size() * sizeof(SkvSlot));
    for (int q = 0; q < kOwned; ++q) up.add(off[q], n_state[q], n_write * 4);
    const int rc = up.up(st);
    if (rc) return rc;
    if (nb_old > live) {
      const size_t n = nb_old - live;
      fill_planes_kernel<<<grid_for(n * SKV_CTR_FIELDS, 256), 256, 0, st>>>(t->dev.ctr, plane, live, n, SKV_CTR_FIELDS);
      fill_u32_kernel<<<grid_for(n, 256), 256, 0, st>>>(t->dev.epoch + live, n, 0u);
      SKV_HIP(hipGetLastError());
    }
    SKV_HIP(hipStreamSynchronize(st));
    return SKV_OK;
  };
  rc = write_back();
  if (rc) {
    for (size_t i = moved.size(); i-- > 0;) move_block((size_t)moved[i].second, (size_t)m->nodes[moved[i].first].first, (size_t)m->nodes[moved[i].first].n_blocks);
    return rc;
  }
  for (size_t i = 0; i < d0; ++i) id_map[i] = (int32_t)i;
  std::copy_n(new_id, n_id, id_map + d0);
  std::fill_n(id_map + d1, nin_old - d1, -1);
  m->tok.resize(live * 16); m->page.resize(live); m->canon.resize(live); m->vis.resize(live); m->node_of.resize(live);
  m->flat_of.resize(n_ids);
  std::copy_n(n_state[0], n_write, m->vis.begin() + f0);
  std::copy_n(canon, n_canon, m->canon.begin() + canon_lo);
  std::copy_n(flat_of, n_ids - id_lo, m->flat_of.begin() + id_lo);
  for (size_t n = 1; n < m->nodes.size(); ++n) {
    if (new_node[n] < 0) continue;
    const SkvNode& nd = nodes[new_node[n]];
    if (new_node[n] != (int32_t)n || (size_t)nd.first >= f0) std::fill_n(m->node_of.begin() + nd.first, nd.n_blocks, new_node[n]);
  }
  m->nodes.swap(nodes);
  m->slots.swap(slots);
  m->kids.swap(kids);
  m->filled.swap(filled);
  m->parent.swap(parent);
  m->slots_used = m->slots.size();
  t->dev.n_blocks = (int32_t)live;
  t->dev.n_nodes = (int32_t)m->nodes.size() - 1;
  t->n_in_blocks = (int64_t)n_ids;
  if (n_in_blocks_after) *n_in_blocks_after = (int64_t)n_ids;
  return SKV_OK;
}

extern "C" int skv_tree_info(const skv_tree* t, int64_t* n_nodes, int64_t* n_blocks, int64_t* n_in_blocks) {
  if (!t) return SKV_EINVAL;
  if (n_nodes) *n_nodes = t->dev.n_nodes;
  if (n_blocks) *n_blocks = t->host ? t->host->live_blocks : t->dev.n_blocks;
  if (n_in_blocks) *n_in_blocks = t->n_in_blocks;
  return SKV_OK;
}

extern "C" void skv_tree_destroy(skv_tree* t) {
  if (t) delete t->host;
  delete t;
}

extern "C" int skv_counters_read(skv_tree* t, uint32_t* d_hit, uint32_t* d_ucnt, void* stream) {
  if (!t || !d_hit || !d_ucnt) return SKV_EINVAL;
  hipStream_t st = (hipStream_t)stream;
  if (t->n_in_blocks)
    counters_read_kernel<<<grid_for((size_t)t->n_in_blocks, 256), 256, 0, st>>>(t->dev, t->n_in_blocks, d_hit, d_ucnt);
  SKV_HIP(hipGetLastError());
  return SKV_OK;
}

extern "C" int skv_counters_reset(skv_tree* t, void* stream) {
  if (!t) return SKV_EINVAL;
  if (t->dev.n_blocks)
    counters_clear_window_kernel<<<grid_for((size_t)t->dev.n_blocks, 256), 256, 0, (hipStream_t)stream>>>(t->dev);
  SKV_HIP(hipGetLastError());
  return SKV_OK;
}

extern "C" int skv_window_roll(skv_tree* t, const skv_rdr_policy* pol, int32_t* d_n_demoted, void* stream) {
  if (!t || !pol) return SKV_EINVAL;
  if ((pol->direction != 0 && pol->direction != 1) || pol->tau_den == 0 || pol->n_consec == 0) return SKV_EINVAL;
  hipStream_t st = (hipStream_t)stream;
  if (d_n_demoted) fill_u32_kernel<<<1, 64, 0, st>>>((uint32_t*)d_n_demoted, 1, 0u);
  if (t->dev.n_blocks)
    window_roll_kernel<<<grid_for((size_t)t->dev.n_blocks, 256), 256, 0, st>>>(t->dev, *pol, d_n_demoted);
  if (t->host) t->host->vis_stale = true;   // the kernel decides the demotions
  SKV_HIP(hipGetLastError());
  return SKV_OK;
}

extern "C" int skv_promote(skv_tree* t, const int32_t* d_block_ids, int32_t n, void* stream) {
  if (!t || n < 0 || (n > 0 && !d_block_ids)) return SKV_EINVAL;
  if (n) promote_kernel<<<grid_for((size_t)n, 256), 256, 0, (hipStream_t)stream>>>(t->dev, t->n_in_blocks, d_block_ids, n);
  if (n && t->host) t->host->vis_stale = true;   // the ids are in device memory: the host has not seen them
  SKV_HIP(hipGetLastError());
  return SKV_OK;
}

extern "C" int skv_block_state_read(skv_tree* t, uint8_t* d_private, uint32_t* d_hit_pre, uint32_t* d_u_pre,
                                    void* stream) {
  if (!t) return SKV_EINVAL;
  hipStream_t st = (hipStream_t)stream;
  if (t->n_in_blocks && (d_private || d_hit_pre || d_u_pre))
    block_state_read_kernel<<<grid_for((size_t)t->n_in_blocks, 256), 256, 0, st>>>(t->dev, t->n_in_blocks, d_private, d_hit_pre, d_u_pre);
  SKV_HIP(hipGetLastError());
  return SKV_OK;
}
