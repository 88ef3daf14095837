// The body of the bf16 attention kernels (skv_attn.hip): arguments p; kParts, kPlan, kTwo.  No include guard: it is the text of each.
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
