// The body of k_forward_dataflow (S = DfNarrow) and of k_forward_wide (S = DfWide), see dataflow.h, which includes it in each of them.  (As a function that both
// call it comes out of the compiler with more scalar registers parked in vector lanes: five rows of width 896 394 -> 397 us, nine 452 -> 457.)
  const DArgs& a = df_args();
  __shared__ __attribute__((aligned(16))) uint32_t lds[S::LDS_WORDS];
  __shared__ int srow[3 * 16];
  __shared__ uint32_t sact[16 * S::ACT_PITCH];
  __shared__ int sdead;
  if (threadIdx.x == 0) sdead = 0;
  // this launch's number (the kernel that follows a forward on the stream advances the word; nothing in this launch
  // does).  Requested first, looked at after the other start-up loads have been requested.
  const int tag_v = ld_state(a.kv.ctl + 3);
  const u64 state_v = ld_word(a.state);
  uint32_t tag = 0u;
  size_t set = 0;                                          // where this launch's set of words begins
  const int nqkv = (a.nq + 2 * a.nkv) * S::HD, nqd = a.nq * S::HD, L = a.n_layers, np = a.d >> 5;
  const int NU = gridDim.x * 2;
  // items of every phase kind, and the unit that takes item 0 (the kinds with few items go to different workgroups)
  const int n_qkv = (a.nq + 2 * a.nkv) * (S::HD / 32), ntile = (a.rows.R * (a.nq / a.nkv) + 15) >> 4,
            n_att = a.n_seqs * a.nkv * a.n_parts * ntile * S::NH, n_o = np, n_gu = a.ffn >> 4,
            n_lg = (((a.vocab + 15) >> 4) + 1) >> 1;
  const int st = a.small_stride, so = S::WIDE ? a.o_stride : st;
  const int st_lg = 2 * n_lg <= NU ? 2 : 1;               // the head's items: a workgroup each where there are enough (a CU's intake bounds an item's weight stream)
  // (sums go to the first workgroups, which have MLP items; their own stores' acknowledgement comes just before there is something to sum)
  const int s_att = NU - 2 * n_att, s_qkv = (s_att - st * n_qkv + NU) % NU, s_o = (s_qkv - so * n_o + NU) % NU, s_red = 0;
  auto make_qkv = [&](const DArgs& a, int l) {
    const PLayer Y = layer_ptrs(a, l);
    DPhase x = DPhase{};
    x.layer = l; x.A = a.hg + set + (size_t)(2 * l) * a.st_h; x.sq = a.sq + set + (size_t)(2 * l) * a.st_sq;
    x.W0 = Y.wqkv; x.W1 = Y.wqkv; x.N = nqkv; x.K = a.d; x.gs = 1; x.items = n_qkv; x.shift = s_qkv; x.stride = st;
    x.bias = Y.bqkv; x.out = a.q + set + (size_t)l * a.st_q; x.kvn = a.kvn + set + (size_t)l * a.st_kvn;
    x.hint = x.A;
    return x;
  };
  auto make_o = [&](const DArgs& a, int l) {
    const PLayer Y = layer_ptrs(a, l);
    DPhase x = DPhase{};
    x.layer = l;
    x.A = a.attn + set + (size_t)l * a.st_q;
    x.W0 = Y.wo; x.W1 = Y.wo; x.N = a.d; x.K = nqd; x.gs = 1; x.items = n_o; x.shift = s_o; x.stride = so;
    const size_t hi = (size_t)(2 * l);
    x.h_in = a.h + set + hi * a.st_h; x.h_out = a.h + set + (hi + 1) * a.st_h; x.hg_out = a.hg + set + (hi + 1) * a.st_h;
    x.sq_out = a.sq + set + (hi + 1) * a.st_sq;
    x.gain_next = Y.ln2;
    x.hint = a.q + set + (size_t)l * a.st_q;
    return x;
  };
  auto make_swiglu = [&](const DArgs& a, int l) {
    const PLayer Y = layer_ptrs(a, l);
    DPhase x = DPhase{};
    x.layer = l; x.A = a.hg + set + (size_t)(2 * l + 1) * a.st_h; x.sq = a.sq + set + (size_t)(2 * l + 1) * a.st_sq;
    x.W0 = Y.wgate; x.W1 = Y.wup; x.N = a.ffn; x.K = a.d; x.gs = 1; x.items = n_gu; x.shift = 0; x.stride = 1;
    x.hint = a.hg + set + (size_t)(2 * l + 1) * a.st_h;
    return x;
  };
  auto make_head = [&](const DArgs& a) {
    DPhase x = DPhase{};
    x.A = a.hg + set + (size_t)(2 * L) * a.st_h; x.sq = a.sq + set + (size_t)(2 * L) * a.st_sq;
    x.W0 = a.head; x.W1 = a.head; x.N = a.vocab; x.K = a.d; x.gs = 1; x.items = n_lg; x.shift = 0; x.stride = st_lg; x.logits = a.logits;
    return x;
  };
  // which phase kinds this workgroup has a round-0 item in
  auto has = [&](int u, int shift, int items, int stride = 1) { return df_item_of_unit(u, shift, NU, stride) < items; };
  const int n_red = a.rows.M * ceil_div(a.d, df_sum_cols<SB>());
  const int u0 = blockIdx.x * 2, u1 = u0 + 1;
  const bool g_q = has(u0, s_qkv, n_qkv, st) || has(u1, s_qkv, n_qkv, st) || st * n_qkv > NU,
             g_a = has(u0, s_att, n_att, 2),                  // (an attention item has the workgroup)
             g_o = has(u0, s_o, n_o, so) || has(u1, s_o, n_o, so), g_g = (int)blockIdx.x < a.g_mlp,
             g_r = df_item_of_unit((int)blockIdx.x, s_red >> 1, (int)gridDim.x) < n_red || n_red > (int)gridDim.x, g_l = has(u0, 0, n_lg, st_lg) || has(u1, 0, n_lg, st_lg) || st_lg * n_lg > NU;

  DF_STAMP(1);
  df_reserve_blocks(a, tag_v, blockIdx.x == 0);
  // What the launch needs of the cache state (none of it changes during the launch): the waves' attention items, and
  // per row its position and whether it is active.
  __shared__ int sblk[DF_ONE_CHUNKS * 4];
  const DAttItem ait = df_att_item<S>(a, df_item_of_unit(u0, s_att, NU, 2), ntile, sblk);
  if ((g_q || g_a) && threadIdx.x < a.rows.M) {           // the QKV epilogue and the attention masks use them
    const int m = threadIdx.x, brel = m / a.rows.R, j = m - brel * a.rows.R, seq = a.rows.seq0 + brel;
    const int len = ld_state(a.kv.len + seq);
    const int npend = a.pcap ? ld_state(a.kv.n_pend + seq) : 0;
    const int off = a.pcap - npend;
    srow[m] = j < off ? len : len + (j - off);
    srow[16 + m] = j < off ? 0 : 1;
  }
  tag = (uint32_t)__builtin_amdgcn_readfirstlane(tag_v);
  if (!df_tag_ok(tag)) {                                   // numbering exhausted: do nothing; the host must clear the workspace
    if (blockIdx.x == 0 && threadIdx.x == 0) __hip_atomic_fetch_or(a.bar + 64, DEV_ERR_TAGS, __ATOMIC_RELAXED, AG);
    return;
  }
  // The set of words: the other one than the last launch's.  (The state may already be this launch's: then the launch has gone all its way
  // but for workgroups without an item in the layers, such as this one.)
  const uint32_t last_tag = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)state_v), last = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(state_v >> 32));
  const uint32_t which = last_tag == tag ? last & 1u : ~last & 1u;
  const int old_rows = last_tag == tag ? 0 : (int)(last >> 1);
  set = which * a.st_set;
  df_embed_phase<df_sq_cols<SB>()>(a, set);
  if (g_q && threadIdx.x < a.rows.M) {                    // the QKV epilogue appends keys and values: block of each row's position
    u64 w = ld_word(a.rowblk + threadIdx.x);
    for (long spins = 0; (uint32_t)(w >> 32) != tag; w = ld_word(a.rowblk + threadIdx.x)) {
      if (++spins > DF_SPIN_LIMIT || ((spins & 63) == 0 && __hip_atomic_load(a.bar + 64, __ATOMIC_RELAXED, AG) != 0)) {
        __hip_atomic_store(a.bar + 64, 1u, __ATOMIC_RELAXED, AG);
        w = 0xFFFFFFFFull;                                 // no block: the row is not appended, every later wait sees the flag
        break;
      }
      __builtin_amdgcn_s_sleep(1);
    }
    srow[32 + threadIdx.x] = (int)(uint32_t)w;
  }
  __syncthreads();
  df_loads_done();
  DF_STAMP(0);
  for (int l = 0; l < L; ++l) {
    const int s0 = 2 + l * 10;
    if (g_q) {
      const DArgs& a = df_args();
      const DPhase cur = make_qkv(a, l);
      if (df_gemm_phase<PE_QKV, SB, S>(a, cur, lds, srow, &sdead, s0)) return;
    }
    if (g_a) {
      const DArgs& a = df_args();
      if (df_attn_phase<SB, S>(a, tag, set, l, ait, lds, sblk, srow, &sdead, s0 + 2)) return;
    }
    if (g_o) {
      const DArgs& a = df_args();
      const DPhase cur = make_o(a, l);
      if (df_gemm_phase<PE_RESID, SB, S>(a, cur, lds, srow, &sdead, s0 + 4)) return;
    }
    auto clear = [&]() {
      const DArgs& a = df_args();
      if (g_r && l > 0) df_clear_partials<df_sum_cols<SB>(), S>(a, a.part + (size_t)((l - 1) & 1) * a.st_part, s_red);
      if (g_g) df_clear_layer<S>(a, (which ^ 1u) * a.st_set, old_rows, l);
    };
    if (!g_g) {
      clear();
    } else {
      const DArgs& a = df_args();
      const DPhase cur = make_swiglu(a, l);
      const float* part = a.part + (size_t)(l & 1) * a.st_part;
      if constexpr (S::WIDE) {
        if (df_mlp_wide<SB, S>(a, cur, layer_ptrs(a, l).wdown, part, clear, lds, sact, &sdead, s0 + 6)) return;
      } else {
        if (df_mlp_phase<SB, S>(a, cur, layer_ptrs(a, l).wdown, part, clear, lds, sact, &sdead, s0 + 6)) return;
      }
    }
    if (g_q && g_r && l + 1 < L) {
      const DArgs& a = df_args();
      df_touch_weights<S>(a, make_qkv(a, l + 1));
    }
    if (g_r) {
      const DArgs& a = df_args();
      const size_t hi = (size_t)(2 * l + 1);
      const float* gain_next = l + 1 < L ? layer_ptrs(a, l + 1).ln1 : a.final_norm;
      if (df_reduce_phase<df_sum_cols<SB>(), S>(a, a.part + (size_t)(l & 1) * a.st_part, a.h + set + hi * a.st_h, a.h + set + (hi + 1) * a.st_h,
                          a.hg + set + (hi + 1) * a.st_h, a.sq + set + (hi + 1) * a.st_sq, gain_next, s_red, lds, &sdead, s0 + 8)) return;
    }
  }
  if (a.with_head && g_l) {
    const DArgs& a = df_args();
    const DPhase cur = make_head(a);
    if (df_gemm_phase<PE_LOGITS, SB, S>(a, cur, lds, srow, &sdead, 2 + L * 10)) return;
  }
  if (g_r) {
    const DArgs& a = df_args();
    df_clear_partials<df_sum_cols<SB>(), S>(a, a.part + (size_t)((L - 1) & 1) * a.st_part, s_red);
  }
  // (workgroup 0 sums partials of every MLP item: those have all begun long ago)
  if (blockIdx.x == 0 && threadIdx.x == 0)
    __hip_atomic_store(a.state, (u64)tag | (u64)((uint32_t)a.rows.M << 1 | which) << 32, __ATOMIC_RELAXED, AG);
