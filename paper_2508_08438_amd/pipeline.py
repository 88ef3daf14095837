"""Device-resident state of one workload and the sequence of library calls that makes one pass
of the path.  Only buffer management and calls into `binding`; no arithmetic of the method."""
from __future__ import annotations

import threading

import numpy as np
import torch

from . import binding as skv
from .inputs import BLOCK, Workload


def _tiled_from_host(chunk: torch.Tensor, n_rows: int, device) -> torch.Tensor:
    """[n_rows, ...] device tensor filled with repetitions of a host chunk: host-to-device copies only."""
    out = torch.empty((n_rows,) + tuple(chunk.shape[1:]), dtype=chunk.dtype, device=device)
    step = chunk.shape[0]
    for lo in range(0, n_rows, step):
        hi = min(n_rows, lo + step)
        out[lo:hi].copy_(chunk[: hi - lo])
    return out


# K and V bytes from which a step copies them on a stream of its own beside the attention.  The two queues' waits cost about
# 15 us, attention slows by a third of the copy's time, and offsets and counters take launches of their own again: us a pass, beside /
# in one call: 12 MB behind one request 59 / 37.5; 98 MB, 3 of 8 rows, 85 / 81; 154 MB, 7 of up to 137, 110 / 114; 250 MB, 93 of 46, 145 /
# 175; 3.3 GB, 32 requests, 6865 / 7524.  Of 70 steps of 65 MB to 1.4 GB, attention from 26 us to 1.2 ms, one call is the faster for 18 of
# the 20 below the line (the others by 1 and 4 %), two streams for 45 of the 50 above it (the others by up to 6 %).
GATHER_BESIDE_BYTES = 128 << 20

# Bytes a pool and a page from which that form of the copy is the faster one alone (4096 pages of 32 KB 101 -> 93 us): a session's staging
# is as large as what it holds.
GATHER_ALONE_BYTES, GATHER_ALONE_PAGE = 48 << 20, 16384

# One stream per device for these copies, whatever the number of sessions: streams are dealt to four hardware queues, and a copy on
# the queue of the attention's own stream runs behind it (24 requests behind 1700 keys, on nine streams one after the other: 260
# to 264 us, on the sixth 296).  A capture takes a stream of the session's own.  Neither is of torch's pool (binding.OwnStream).
_copy_streams = {}
_copy_lock = threading.Lock()


def _copy_stream(device):
    with _copy_lock:
        if device not in _copy_streams:
            _copy_streams[device] = skv.OwnStream(device)
            _copy_streams[device].record_event()      # its queue is there before the first pass
        return _copy_streams[device]


class Session:
    """host_fill=True builds every device buffer from host memory with plain copies, so that no torch device
    kernel runs in the process (for hardware-counter runs, which must see the library's kernels only).  Pools and
    Q/K/V then hold repetitions of one host-generated chunk: same shapes and access pattern, other values.
    kpool / vpool: pools of another session of the same configuration and seed, shared instead of filled again."""

    def __init__(self, w: Workload, device="cuda:0", with_kv=True, gather=True, host_fill=False, kpool=None,
                 vpool=None):
        self.w, self.device, self.do_gather, self.host_fill = w, torch.device(device), gather, host_fill
        dev = self.device
        a = w.attn
        self.desc = skv.attn_desc(a.n_q_heads, a.n_kv_heads, a.head_dim, a.dtype, a.scale)
        self.tree = skv.skv_tree_build(w.seq_tokens, w.seq_off, w.blk_sensitive, w.blk_owner, w.blk_page,
                                       w.n_tenants, w.n_pages, device=dev)
        self.req_off = torch.from_numpy(w.req_off).to(dev)
        self.req_tokens = torch.from_numpy(w.req_tokens).to(dev)
        self.req_tenant = torch.from_numpy(w.req_tenant).to(dev)
        R = w.n_req
        self.max_blocks = max(w.max_blocks, 1)
        self.matched_len = torch.zeros(R, dtype=torch.int32).to(dev)
        self.page_table = torch.full((R, self.max_blocks), -1, dtype=torch.int32).to(dev)
        self.q_off = torch.zeros(R + 1, dtype=torch.int32).to(dev)
        self.ctx_off = torch.zeros(R + 1, dtype=torch.int64).to(dev)
        self.kpool, self.vpool = kpool, vpool
        if with_kv and kpool is None:  # match-only sessions never touch the pools
            shape = (w.n_pages, BLOCK, a.n_kv_heads, a.head_dim)
            if host_fill:
                n = min(w.n_pages, 2048)
                self.kpool = _tiled_from_host(w.pool_pages("k", 0, n), w.n_pages, dev)
                self.vpool = _tiled_from_host(w.pool_pages("v", 0, n), w.n_pages, dev)
            else:
                self.kpool = torch.empty(shape, dtype=a.torch_dtype, device=dev)
                self.vpool = torch.empty(shape, dtype=a.torch_dtype, device=dev)
                w.fill_pool("k", self.kpool)
                w.fill_pool("v", self.vpool)
        self.q = None
        self.side = self.side_capture = None     # streams of a copy beside the attention

    # -- one-off: lay out Q / K_new / V_new for the suffixes this workload's match leaves uncached
    def prepare(self):
        w, dev, a = self.w, self.device, self.w.attn
        skv.skv_counters_reset(self.tree)
        skv.skv_match(self.tree, self.req_off, self.req_tokens, self.req_tenant, self.max_blocks,
                      self.matched_len, self.page_table)
        torch.cuda.synchronize(dev)
        ml = self.matched_len.cpu().numpy()
        self.host_matched_len = ml
        n_ctx = max(int(ml.sum()), BLOCK)
        if self.host_fill:
            total = int((np.diff(w.req_off) - ml).sum())
            n = min(max(total, 1), 4096)
            self.q = _tiled_from_host(w.token_rows("q", 0, n), total, dev)
            self.knew = _tiled_from_host(w.token_rows("k", 0, n), total, dev)
            self.vnew = _tiled_from_host(w.token_rows("v", 0, n), total, dev)
            self.out = torch.empty_like(self.q)
            self.kctx = torch.empty((n_ctx, a.n_kv_heads, a.head_dim), dtype=a.torch_dtype, device=dev)
            self.vctx = torch.empty_like(self.kctx)
        else:
            self.q = w.suffix_rows("q", ml, dev)
            self.knew = w.suffix_rows("k", ml, dev)
            self.vnew = w.suffix_rows("v", ml, dev)
            self.out = torch.zeros_like(self.q)
            self.kctx = torch.zeros((n_ctx, a.n_kv_heads, a.head_dim), dtype=a.torch_dtype, device=dev)
            self.vctx = torch.zeros_like(self.kctx)
        page = BLOCK * a.n_kv_heads * a.head_dim * self.kctx.element_size()
        self.large_copy = page >= GATHER_ALONE_PAGE and self.kctx.numel() * self.kctx.element_size() >= GATHER_ALONE_BYTES
        self.records = torch.empty_like(self.page_table)     # of the matched blocks, between the kernels of a step
        nbytes = skv.skv_prefill_attn_workspace_size(self.desc, w.n_req, self.q.shape[0])
        self.workspace = torch.empty(nbytes, dtype=torch.uint8, device=dev)
        copied = 2 * self.kctx.numel() * self.kctx.element_size()
        if self.do_gather and a.dtype == "bf16" and copied >= GATHER_BESIDE_BYTES:   # (fp32 attention leaves no registers)
            self.side, self.side_capture = _copy_stream(self.q.device), skv.OwnStream(dev)
        skv.skv_counters_reset(self.tree)

    # -- the individual stages (each only enqueues on the current stream)
    def match(self):
        skv.skv_counters_reset(self.tree)
        skv.skv_match(self.tree, self.req_off, self.req_tokens, self.req_tenant, self.max_blocks,
                      self.matched_len, self.page_table)
        skv.skv_suffix_offsets(self.req_off, self.matched_len, self.q_off)

    def gather(self, stream=None, beside=False):
        skv.skv_gather_kv(self.desc, self.kpool, self.vpool, self.matched_len, self.page_table,
                          self.max_blocks, self.ctx_off, self.kctx, self.vctx, stream=stream,
                          beside=beside or self.large_copy)

    def attention(self):
        skv.skv_prefill_attn(self.desc, self.q, self.knew, self.vnew, self.q_off, self.kpool, self.vpool,
                             self.matched_len, self.page_table, self.max_blocks, self.out, self.workspace)

    def _pass(self):
        """Gather and attention both read the match's results and neither the other's: a large copy runs on a stream of its own
        beside the attention (the current stream waits for it before this returns, also where attention() raises); what is
        smaller, the suffix offsets and the counters of the lookup share the attention's call."""
        main = torch.cuda.current_stream() if self.side else None
        if self.do_gather and (main is None or main.device != self.side.device):
            left = skv.skv_match_window(self.tree, self.req_off, self.req_tokens, self.req_tenant, self.max_blocks, self.matched_len,
                                        self.page_table, self.records)
            return skv.skv_prefill_step(self.desc, self.req_off, self.q, self.knew, self.vnew, self.q_off, self.kpool, self.vpool,
                                        self.matched_len, self.page_table, self.max_blocks, self.out, self.ctx_off, self.kctx,
                                        self.vctx, self.workspace, tree=self.tree, req_tenant=self.req_tenant,
                                        records=self.records if left else None)
        self.match()
        if not self.do_gather:
            return self.attention()
        side = self.side_capture if torch.cuda.is_current_stream_capturing() else self.side
        matched = main.record_event()
        try:
            self.attention()      # first: it is what the copy has to fit beside
        finally:
            side.wait_event(matched)
            self.gather(stream=side, beside=True)
            main.wait_stream(side)

    def step(self):
        if self.q is None:
            self.prepare()
        self._pass()
        return {"matched_len": self.matched_len, "page_table": self.page_table, "q_off": self.q_off,
                "ctx_off": self.ctx_off, "out": self.out, "kctx": self.kctx, "vctx": self.vctx}

    # -- the same pass recorded once as a HIP graph and replayed: the calls of match / gather / attention only
    #    enqueue kernels on the stream they are given (no allocation, no memset, no synchronisation)
    def capture_step(self):
        if self.q is None:
            self.prepare()
        self.step()                       # everything loaded and warm before the capture
        torch.cuda.synchronize(self.device)
        self.graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(self.graph):
            self._pass()
        return self.graph

    def replay(self):
        self.graph.replay()

    def counters(self):
        n = self.w.n_in_blocks
        hit = torch.zeros(max(n, 1), dtype=torch.int32).to(self.device)
        ucnt = torch.zeros(max(n, 1), dtype=torch.int32).to(self.device)
        skv.skv_counters_read(self.tree, hit, ucnt)
        torch.cuda.synchronize(self.device)
        return hit[:n].cpu().numpy().view(np.uint32), ucnt[:n].cpu().numpy().view(np.uint32)

    def host_pools(self, page_table):
        """CPU copies of the pools holding the pages a page table references (others zero)."""
        w, a = self.w, self.w.attn
        pages = np.unique(page_table[page_table >= 0])
        shape = (w.n_pages, BLOCK, a.n_kv_heads, a.head_dim)
        kpool = torch.zeros(shape, dtype=a.torch_dtype)
        vpool = torch.zeros(shape, dtype=a.torch_dtype)
        w.fill_pool("k", kpool, pages)
        w.fill_pool("v", vpool, pages)
        return kpool, vpool
