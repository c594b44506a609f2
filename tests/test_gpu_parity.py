"""GPU parity tests: the HIP path (through the C ABI) against the CPU oracle, element by element."""
import numpy as np
import pytest
import torch

import synth_inputs as si

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2505_15380_amd as pkg
    pkg.load_library()                      # fail loudly if the HIP library is missing


def grid24(a):
    return (np.floor(np.asarray(a) * (1 << 24)) / (1 << 24)).astype(np.float32)


# ------------------------------------------------------------------------------ acceptance alone (Eq. 5-6)
@pytest.mark.parametrize("V,K,B", [(7, 1, 3), (512, 4, 8), (6564, 4, 4), (6564, 12, 2), (1000, 0, 5), (257, 15, 3),
                                   (8192, 2, 2), (8193, 2, 2), (16384, 3, 2)])   # both unrolled sizes of the sampler kernels
@pytest.mark.parametrize("beta", [0.0, 0.4])
def test_decisions_bit_exact_given_probabilities_and_uniforms(V, K, B, beta):
    import paper_2505_15380_amd as ssd
    from oracle.accept import accept_canonical
    rng = np.random.default_rng(V * 31 + K)
    for trial in range(6):
        alpha = [0.05, 0.5, 5.0][trial % 3]
        pt = si.make_probs(rng, B * (K + 1), V, alpha, zeros=0.3 * (trial % 2)).reshape(B, K + 1, V)
        pd = si.make_probs(rng, max(B * K, 1), V, alpha).reshape(-1, V)[:B * K].reshape(B, K, V)
        if trial == 4 and K > 0:
            pd[:, 0] = pt[:, 0]             # draft == target on the first position: ratio exactly 1
        x = rng.integers(0, V, size=(B, K)).astype(np.int32)
        if K:
            for b in range(B):              # mostly plausible draft tokens (drawn from pd)
                for i in range(K):
                    if rng.random() < 0.8:
                        q = pd[b, i].astype(np.float64)
                        x[b, i] = rng.choice(V, p=q / q.sum())
        u = grid24(rng.random((B, K + 1)))
        if trial == 5:
            u[:, :K] = grid24(1 - 2.0 ** -24)   # the largest uniform
        n, nxt, fl = ssd.ssd_verify_from_probs(torch.from_numpy(pt).cuda(), torch.from_numpy(pd).cuda(),
                                               torch.from_numpy(x).cuda(), torch.from_numpy(u).cuda(), beta)
        n, nxt, fl = n.cpu().numpy(), nxt.cpu().numpy(), fl.cpu().numpy()
        for b in range(B):
            want = accept_canonical(pt[b], pd[b], list(x[b]), list(u[b, :K]), u[b, K], beta)
            assert (int(n[b]), int(nxt[b]), bool(fl[b])) == want, (trial, b, want)


def test_decisions_degenerate_rows():
    import paper_2505_15380_amd as ssd
    from oracle.accept import accept_canonical
    V = 300
    # zero residual (falls back to pt), subnormal probabilities, one-hot rows, pd(x) = 0
    pt = np.zeros((4, 2, V), np.float32)
    pd = np.zeros((4, 1, V), np.float32)
    x = np.zeros((4, 1), np.int32)
    pt[0, 0, :3] = [0.25, 0.25, 0.5]; pd[0, 0, :3] = [0.5, 0.5, 1.0]; x[0, 0] = 2; pt[0, 1, 7] = 1
    pt[1, 0, 0] = 1e-41; pt[1, 0, 1] = 1; pd[1, 0, 0] = 4e-41; pd[1, 0, 1] = 1; x[1, 0] = 0; pt[1, 1, 9] = 1
    pt[2, 0, 5] = 1; pd[2, 0, 6] = 1; x[2, 0] = 6; pt[2, 1, 11] = 1
    pt[3, 0, 5] = 1; pd[3, 0, 6] = 1; x[3, 0] = 5; pt[3, 1, 299] = 1          # pd(x) = 0 -> accepted
    for r0 in (0.1, 0.2, 0.3, 0.9):
        u = grid24(np.array([[r0, 0.6]] * 4))
        n, nxt, fl = ssd.ssd_verify_from_probs(torch.from_numpy(pt).cuda(), torch.from_numpy(pd).cuda(),
                                               torch.from_numpy(x).cuda(), torch.from_numpy(u).cuda(), 0.0)
        for b in range(4):
            want = accept_canonical(pt[b], pd[b], list(x[b]), [u[b, 0]], u[b, 1], 0.0)
            assert (int(n[b]), int(nxt[b]), bool(fl[b])) == want, (r0, b, want)


@pytest.mark.parametrize("V", [3, 1024, 1025, 6564, 8192, 8193, 9000, 16383])
def test_draw_reaches_every_index_at_both_ends_of_a_row(V):
    """A thread draws from a contiguous span of indices, and those at the row's end from one that overlaps their neighbours' loads: all the mass
    on one index, as the row itself (no drafts) and as the residual of a rejected draft."""
    import paper_2505_15380_amd as ssd
    j = np.unique(np.concatenate([np.arange(min(V, 20)), np.arange(max(V - 40, 0), V)]))
    j = j[j > 0]                             # (the draft's token is 0)
    B = len(j)
    pt, pd = np.zeros((B, 2, V), np.float32), np.zeros((B, 1, V), np.float32)
    pt[np.arange(B), 0, j] = 1.0
    pd[:, 0, 0] = 1.0
    for u in (0.0, 0.5, 1.0 - 2.0 ** -24):
        uu = grid24(np.full((B, 2), u))
        uu[:, 0] = 0.5
        n, nxt, _ = ssd.ssd_verify_from_probs(torch.from_numpy(pt).cuda(), torch.from_numpy(pd).cuda(), torch.zeros(B, 1, dtype=torch.int32).cuda(),
                                              torch.from_numpy(uu).cuda(), 0.0)
        assert (n.cpu().numpy() == 0).all() and (nxt.cpu().numpy() == j).all(), u
        n, nxt, _ = ssd.ssd_verify_from_probs(torch.from_numpy(pt[:, :1].copy()).cuda(), None, None, torch.from_numpy(uu[:, 1:].copy()).cuda(), 0.0)
        assert (nxt.cpu().numpy() == j).all(), u


# ------------------------------------------------------------------------------ warp + softmax alone
@pytest.mark.parametrize("V", [512, 6564, 1000, 8192, 8193, 16384])
def test_warp_probs_against_oracle(V):
    import paper_2505_15380_amd as ssd
    from oracle.warp import warp_probs
    rng = np.random.default_rng(V)
    z = (rng.standard_normal((6, V)) * 2).astype(np.float32)
    z[1, 100:140] = z[1, 7]                  # a long tie that straddles top-k cuts
    z[2, :] = 0.5                            # all equal
    z[3, 5] = z[3].max(); z[3, 3] = z[3].max()
    for kw in (dict(), dict(temperature=0.8), dict(top_k=25), dict(top_k=25, temperature=0.7), dict(top_k=1),
               dict(greedy=True), dict(top_k=V - 1), dict(top_k=V + 5)):
        got = ssd.ssd_warp_probs(torch.from_numpy(z).cuda(), ssd.sample_config(**kw)).cpu().numpy()
        ref = warp_probs(z.astype(np.float64), kw.get("temperature", 1.0), kw.get("top_k", 0), kw.get("greedy", False))
        assert ((got > 0) == (ref > 0)).all(), kw           # the kept set is exact, ties included
        assert np.abs(got - ref).max() < 1e-6, kw
        assert np.abs(got.sum(axis=1) - 1).max() < 1e-5


@pytest.mark.parametrize("k", [2, 127, 128, 129, 255, 512, 513, 1024])
def test_top_k_cut_at_the_edges_of_the_candidate_set(k):
    """k on both sides of the sizes at which the search for the cut stops, with ties that are longer than any candidate
    set, peaked rows and rows of few distinct values."""
    import paper_2505_15380_amd as ssd
    from oracle.warp import warp_probs
    V = 6564
    rng = np.random.default_rng(k)
    z = rng.standard_normal((7, V)).astype(np.float32)
    z[1] = np.round(z[1])                                    # a dozen distinct values
    z[2, 200:1500] = z[2].max() + 1.0                        # 1300 entries tie at the maximum
    z[3, 200:1500] = np.sort(z[3])[-20]                      # ... and just below it
    z[4, 77] = 40.0
    z[5] = -np.abs(z[5])
    z[6] = np.where(rng.random(V) < 0.5, 0.0, -0.0).astype(np.float32) + np.float32(1e-30) * z[6]
    got = ssd.ssd_warp_probs(torch.from_numpy(z).cuda(), ssd.sample_config(top_k=k)).cpu().numpy()
    ref = warp_probs(z.astype(np.float64), 1.0, k, False)
    assert ((got > 0) == (ref > 0)).all()
    assert np.abs(got - ref).max() < 1e-6


@pytest.mark.parametrize("V,k", [(5, 2), (600, 200), (6564, 25), (6564, 3300), (9000, 513)])
def test_top_k_cut_among_zeros_of_both_signs(V, k):
    """-0 and +0 are one value: where the cut falls among them, the lower indices stay.  And subnormal numbers are not zeros."""
    import paper_2505_15380_amd as ssd
    from oracle.warp import warp_probs
    rng = np.random.default_rng(V + k)
    z = np.where(rng.random((4, V)) < 0.5, np.float32(0.0), np.float32(-0.0))
    z[1] = np.where(rng.random(V) < 0.5 * k / V, np.float32(1.0), z[1])
    z[2] = np.where(rng.random(V) < 0.3, np.float32(-1.0), z[2])
    z[3] = rng.integers(-3, 4, V).astype(np.float32) * np.float32(1e-41)
    got = ssd.ssd_warp_probs(torch.from_numpy(z).cuda(), ssd.sample_config(top_k=k)).cpu().numpy()
    ref = warp_probs(z.astype(np.float64), 1.0, k, False)
    assert ((got > 0) == (ref > 0)).all()
    assert np.abs(got - ref).max() < 1e-6


@pytest.mark.parametrize("V,k", [(2, 1), (9, 5), (60, 25), (260, 50), (1030, 25), (6564, 25), (6564, 50), (6564, 128), (9000, 128), (16384, 300)])
def test_top_k_cut_where_large_entries_share_their_threads(V, k):
    """The kernel bounds the cut by the maxima of 128 groups of entries (i % 1024 // 8).  Rows whose large entries lie in one group,
    in few groups, in exactly k groups, one per group, or are infinite; and vocabularies with fewer groups than k."""
    import paper_2505_15380_amd as ssd
    from oracle.warp import warp_probs
    rng = np.random.default_rng(V + k)
    z = rng.standard_normal((7, V)).astype(np.float32)
    group = np.arange(V) % 1024 // 8
    z[1, group == group.max() // 2] += 9.0
    z[2, group < 5] += 9.0
    z[3, group < k] += 9.0
    z[4, group >= min(k, 128) - 1] -= 20.0
    z[5, ::3] = -np.inf
    z[6] = np.sort(z[6])
    got = ssd.ssd_warp_probs(torch.from_numpy(z).cuda(), ssd.sample_config(top_k=k, temperature=0.9)).cpu().numpy()
    ref = warp_probs(z.astype(np.float64), 0.9, k, False)
    assert np.abs(got - ref).max() < 1e-6
    kept = ref > 1e-30                       # (what lies far below the maximum underflows in single precision)
    assert (got[kept] > 0).all() and (got[ref == 0] == 0).all()


# ------------------------------------------------------------------------------ the whole verify step
@pytest.mark.parametrize("beta", [0.0, 0.4])
def test_tiny_fp32_verify_parity(beta):
    from tests.parity import run_verify_parity
    r = run_verify_parity("tiny", steps=16, K=4, beta=beta, atol_logits=1e-5, atol_probs=1e-5)
    assert len(set(r["accepted"])) > 1       # both accepts and rejections were exercised


def test_mini_bf16_verify_parity():
    from tests.parity import run_verify_parity
    r = run_verify_parity("mini", steps=8, K=4, beta=0.2, atol_logits=2e-2, atol_probs=2e-2)
    assert r["dlogits"] > 0


@pytest.mark.parametrize("K", [0, 1, 7, 12])
def test_mini_bf16_other_draft_lengths(K):
    from tests.parity import run_verify_parity
    run_verify_parity("mini", steps=3, K=K, beta=0.0, atol_logits=2e-2, atol_probs=2e-2, n_prefix=70)


def test_tiny_topk_temperature_and_greedy():
    from tests.parity import run_verify_parity
    run_verify_parity("tiny", steps=4, K=3, beta=0.0, atol_logits=1e-5, atol_probs=1e-5, temperature=0.7, top_k=25)
    run_verify_parity("tiny", steps=4, K=3, beta=0.0, atol_logits=1e-5, atol_probs=1e-5, greedy=True)


# ---- operator-by-operator forward: edges of row tiles, column tiles, k-tiles, chunks and parts ----------------------
@pytest.mark.parametrize("dtype,hd,groups,n_prefix,B,K", [
    ("fp32", 32, 1, 2, 1, 0),        # one row, two keys
    ("fp32", 32, 3, 64, 2, 4),       # 15 query rows per key head, a chunk that is just full
    ("fp32", 64, 2, 509, 1, 8),      # 18 query rows: two tiles; new positions in a ninth chunk (second round of a wave)
    ("fp32", 128, 1, 130, 3, 6),     # head size with half the waves; 21 rows: two row tiles
    ("fp32", 32, 2, 1030, 1, 2),     # more chunks than one part of the attention has
    ("fp32", 64, 2, 2044, 1, 4),     # rows on both sides of the end of a second part, 16 rows of a tile in one of them
    ("fp32", 128, 3, 508, 2, 6),     # the smaller parts of head size 128
    ("bf16", 128, 3, 2, 1, 0),       # one row
    ("bf16", 64, 7, 60, 17, 0),      # 17 rows: one more than a tile
    ("bf16", 64, 2, 129, 4, 15),     # 64 rows; a prompt of 128 cached positions in one chunk of rows
    ("bf16", 128, 2, 66, 5, 12),     # 65 rows
    ("bf16", 64, 1, 514, 1, 15),     # prompt in 513 rows: one more than take the norm in the projection's epilogue
    ("bf16", 128, 3, 1025, 1, 4)])   # prompt in 1024 rows, 17 chunks of keys
def test_forward_at_the_edges_of_tiles(dtype, hd, groups, n_prefix, B, K):
    """Widths of 9, 25 and odd numbers of tiles, a ragged vocabulary: cache contents after the prompt (one forward of
    n_prefix - 1 rows) and two verifications of B x (K + 1) rows against the oracle."""
    from tests.parity import Pair, verify_parity_step
    shape = dict(n_layers=2, d_model=288, n_q_heads=2 * groups, n_kv_heads=2, head_dim=hd, d_ffn=800, vocab=333,
                 n_embed=340, dtype=dtype, qkv_bias=1, rope_base=1.0e5, rms_eps=1e-6)
    atol = 2e-5 if dtype == "fp32" else 2e-2
    rows = min(max(n_prefix - 1, K + 1), 1024 // B)
    pair = Pair(None, 77, n_prefix + 2 * (K + 1) + 16, max_seqs=B, max_rows=rows, shape=shape)
    rng = np.random.default_rng(78)
    for b in range(B):
        pair.prefill(b, rng.integers(0, 340, max(2, n_prefix - 5 * b)))
        pair.check_state(b, atol)
    for s in range(2):
        verify_parity_step(pair, dict(beta=0.3, seed=79), K, s, rng, atol, atol, seqs=range(B))
    for b in range(B):
        pair.check_state(b, atol)
    pair.check_free_stack()


@pytest.mark.parametrize("dtype,d,hd,ffn,K", [
    ("fp32", 32, 32, 32, 8),         # two k-steps for four waves; nine rows
    ("fp32", 32, 64, 96, 15),
    ("fp32", 64, 128, 32, 8),
    ("fp32", 96, 32, 160, 8),
    ("bf16", 32, 64, 32, 8),         # one pair of output tiles for the eight waves of the barrier-free kernel
    ("bf16", 32, 64, 64, 15),
    ("bf16", 96, 64, 1056, 8),
    ("bf16", 64, 64, 32, 3),
    ("bf16", 32, 128, 32, 8),        # one launch per operator
    ("bf16", 96, 32, 160, 8)])
def test_narrowest_models(dtype, d, hd, ffn, K):
    """The smallest widths that a model may have: a prompt in one forward of 25 rows and two verifications of 4, 9 or 16
    rows against the oracle."""
    from tests.parity import Pair, verify_parity_step
    shape = dict(n_layers=2, d_model=d, n_q_heads=2, n_kv_heads=1, head_dim=hd, d_ffn=ffn, vocab=41, n_embed=43, dtype=dtype,
                 qkv_bias=1, rope_base=1.0e4, rms_eps=1e-6)
    atol = 2e-5 if dtype == "fp32" else 2e-2
    pair = Pair(None, 81, 26 + 2 * (K + 1) + 16, max_rows=25, shape=shape)
    rng = np.random.default_rng(82)
    pair.prefill(0, rng.integers(0, 43, 26))
    pair.check_state(0, atol)
    for s in range(2):
        verify_parity_step(pair, dict(beta=0.3, seed=83), K, s, rng, atol, atol)
        pair.check_state(0, atol)
    pair.check_free_stack()


def check_prompt(shape, rows, seed, tweak=None):
    """A prompt of `rows` positions in one forward with one launch per operator, on two layers of weights with which a tile counts
    (tests.parity.loud_weights), against the oracle with the cache's format.  Keys and values then differ where they round the other
    way, by at most one step of bf16, 2^-7 of the element: no row of a position by more than that of its norm."""
    from tests.parity import Pair, loud_weights
    w = loud_weights(shape, seed)
    if tweak:
        tweak(w)
    pair = Pair(None, 0, rows + 32, max_rows=1024, shape=shape, weights=w, store="bf16")
    pair.prefill(0, np.random.default_rng(seed + 1).integers(0, 43, rows + 1))
    assert pair.kv.last_forward_path() == 1
    pair.check_rows(0, 2.0 ** -7)
    pair.check_state(0, 2.0 ** -4)           # (a step of a value between 8 and 16)
    pair.check_free_stack()


@pytest.mark.parametrize("d,rows", [(32, 65), (96, 80), (544, 64), (544, 65), (1056, 513), (2112, 81), (1056, 961), (1600, 1009), (2464, 769),
                                    (2080, 961), (3104, 961)])
def test_norm_between_the_projections_of_a_prompt(d, rows):
    """The output projection leaves a row's sum of squares in pieces that gate / up adds: one per 16 columns up to 64 rows, above that one
    per pair of tiles or per workgroup - fewer than 16 pieces, ragged, more than 64 (d = 2112), both kernels and every tile of theirs
    (test_launch_plans_cpu.py).  The last 32 columns are made a third of a row's sum or more."""
    def tweak(w):
        for l in range(2):
            w[f"l{l}.wo"][-32:] *= 8.0

    check_prompt(dict(n_layers=2, d_model=d, n_q_heads=2, n_kv_heads=1, head_dim=64, d_ffn=96, vocab=41, n_embed=43, dtype="bf16",
                      qkv_bias=1, rope_base=1.0e4, rms_eps=1e-6), rows, 85, tweak)


@pytest.mark.parametrize("d,ffn,rows", [(32, 96, 65), (64, 8992, 71), (96, 8992, 97), (64, 4896, 250), (32, 8992, 257), (96, 4896, 321),
                                        (32, 8992, 250), (64, 4896, 513), (64, 8992, 449), (1056, 2016, 65), (1056, 2016, 449),
                                        (3616, 96, 897), (4128, 96, 961)])
def test_gate_up_and_down_at_each_tile_of_many_rows(d, ffn, rows):
    """Each tile of the gate / up projection that the estimate picks (in this order: 4 x 8 of k_gemm_block, 5 x 6, 7 x 6, 4 x 10, then
    4 x 8 of k_gemm_tile, 8 x 8, 8 x 10, 8 x 12, 16 x 10; the last four are for down's 4 x 8, 8 x 7, 8 x 8 and 16 x 6; test_launch_plans_cpu.py
    holds the choice), with fewer k-tiles than buffers, a last row tile of one row, and a ragged last column block.  The last 16 of a row's SwiGLU
    columns move its keys and values in the second layer by 1.2 % or more."""
    check_prompt(dict(n_layers=2, d_model=d, n_q_heads=2, n_kv_heads=1, head_dim=64, d_ffn=ffn, vocab=41, n_embed=43, dtype="bf16",
                      qkv_bias=1, rope_base=1.0e4, rms_eps=1e-6), rows, 87)


@pytest.mark.parametrize("nq,nkv,hd,rows", [(2, 1, 64, 513), (15, 3, 64, 1009), (5, 1, 128, 640), (9, 1, 128, 1024)])
def test_qkv_projection_of_more_than_512_rows(nq, nkv, hd, rows):
    """Both of its tiles, 4 x 4 and (336 and 352 workgroups of that) 4 x 8, with last blocks of half a head and of a few rows.  16 dims of
    one query head of a row move its values in the second layer by 5 % or more."""
    check_prompt(dict(n_layers=2, d_model=64, n_q_heads=nq, n_kv_heads=nkv, head_dim=hd, d_ffn=96, vocab=41, n_embed=43, dtype="bf16",
                      qkv_bias=1, rope_base=1.0e4, rms_eps=1e-6), rows, 89)


# d, ffn, query heads, kv heads, rows; {projection: (kernel, row tiles, column slots)} as ssd_gemm_plan names them
@pytest.mark.parametrize("d,ffn,nq,nkv,rows,tiles", [
    (384, 64, 4, 1, 369, {"down": (1, 4, 4), "gate_up": (1, 2, 8), "o": (3, 3, 2), "qkv": (3, 3, 2)}),
    (1792, 256, 9, 1, 66, {"down": (3, 2, 2), "o": (3, 2, 2)}),
    (256, 3072, 5, 1, 161, {"down": (3, 4, 4), "gate_up": (2, 8, 8)}),
    (768, 5760, 4, 1, 65, {"down": (3, 4, 3), "gate_up": (1, 4, 6)}),
    (1792, 64, 4, 1, 641, {"down": (1, 4, 8), "o": (3, 4, 3)}),
    (768, 64, 4, 1, 481, {"o": (3, 2, 3)}),
    (448, 64, 10, 2, 897, {"o": (3, 2, 4), "qkv": (2, 4, 4)}),
    (384, 6400, 5, 1, 65, {"gate_up": (1, 4, 8)}),
    (768, 6400, 6, 1, 130, {"down": (1, 4, 6), "gate_up": (2, 4, 10)}),
    (256, 8960, 4, 1, 129, {"gate_up": (2, 8, 10)}),
    (1792, 64, 7, 1, 433, {"o": (3, 4, 4)}),
    (1792, 64, 7, 1, 577, {"o": (3, 4, 6)}),
    (256, 7680, 4, 1, 257, {"gate_up": (1, 8, 16)}),
    (768, 128, 40, 2, 385, {"qkv": (2, 4, 6)}),
    (1536, 3648, 4, 1, 129, {"down": (2, 8, 6)}),
    (512, 64, 40, 2, 577, {"qkv": (1, 4, 8)}),
    (896, 4864, 4, 1, 1009, {"gate_up": (2, 16, 10), "down": (2, 8, 7)}),
    (288, 8768, 4, 1, 385, {"gate_up": (2, 16, 10)}),
    (320, 8768, 4, 1, 385, {"gate_up": (2, 16, 10), "down": (1, 4, 6)}),
    (352, 8768, 4, 1, 385, {"gate_up": (2, 16, 10)}),
    (2048, 2656, 4, 1, 257, {"down": (2, 8, 7)}),
    (1856, 2944, 4, 1, 385, {"down": (2, 8, 8)}),
    (256, 1824, 4, 1, 17, {"down": (3, 2, 2)}),
    (1088, 1824, 4, 1, 17, {"down": (3, 4, 4)})])
def test_projections_at_the_tiles_of_the_fit(d, ffn, nq, nkv, rows, tiles):
    """The tiles that widths of whole 64 columns and at least eight k-tiles take, each with a ragged last block of rows and, where the
    width allows, of columns; k ranges that leave every number of k-tiles behind the loop.  The large tiles (16 x 10 of gate / up, 8 x 7 and
    8 x 8 of down, in four k-slices) go round their loop twice and more; the last two sizes leave the last of eight slices one k-tile.
    (8 x 12 of gate / up and 8 x 12 of down need full-size models: the batch of the 1.5B shape in test_gpu_fullsize.py.)"""
    import ctypes
    import paper_2505_15380_amd as ssd
    size = {"qkv": (0, (nq + 2 * nkv) * 64, d), "o": (2, d, nq * 64), "gate_up": (3, ffn, d), "down": (4, d, ffn)}
    plan = (ctypes.c_int * 4)()
    for name, want in tiles.items():
        kind, n, k = size[name]
        assert ssd.load_library().ssd_gemm_plan(kind, rows, n, k, 256, plan) == 0 and tuple(plan[:3]) == want, name
    check_prompt(dict(n_layers=2, d_model=d, n_q_heads=nq, n_kv_heads=nkv, head_dim=64, d_ffn=ffn, vocab=41, n_embed=43, dtype="bf16",
                      qkv_bias=1, rope_base=1.0e4, rms_eps=1e-6), rows, 91)


def test_head_of_many_rows():
    """97 sequences x 8 rows: the head in tiles of 16 x 8, with a last block of eight of its 48 row tiles and a ragged last column block
    (test_launch_plans_cpu.py)."""
    from tests.parity import Pair, verify_parity_step
    shape = dict(n_layers=1, d_model=64, n_q_heads=2, n_kv_heads=1, head_dim=64, d_ffn=96, vocab=6564, n_embed=6564, dtype="bf16",
                 qkv_bias=1, rope_base=1.0e4, rms_eps=1e-6)
    B, K = 97, 7
    pair = Pair(None, 93, 32, max_seqs=B, max_rows=K + 1, shape=shape, store="bf16")
    rng = np.random.default_rng(94)
    for b in range(B):
        pair.prefill(b, rng.integers(0, 6564, 2 + b % 9))
    verify_parity_step(pair, dict(beta=0.3, seed=95), K, 0, rng, 4e-3, 4e-3, seqs=range(B))
    assert pair.kv.last_forward_path() == 1
    pair.check_free_stack()


# ---- the barrier-free persistent forward (bf16 shapes, <= 16 rows) ------------------------------------------------
@pytest.mark.gpu
@pytest.mark.parametrize("n_prefix,K", [(250, 4), (254, 12), (600, 4), (1290, 7), (1532, 7)])
def test_mini_bf16_long_prefix_parts_and_boundaries(n_prefix, K):
    """Prefix lengths whose new positions cross a 64-key chunk, one, two and three rounds of chunks per wave, and rows on both
    sides of the 1536 positions up to which a row attends in one part, against the oracle; the barrier-free kernel must be the
    one that ran."""
    from tests.parity import run_verify_parity
    r = run_verify_parity("mini", steps=3, K=K, beta=0.3, atol_logits=2e-2, atol_probs=2e-2, n_prefix=n_prefix)
    assert r["dlogits"] < 2e-2
    assert r["path"] == 3, "the barrier-free persistent kernel did not run"


@pytest.mark.gpu
@pytest.mark.parametrize("n_prefix,K", [(40, 4), (250, 4), (254, 12), (700, 7), (1290, 4), (1500, 3)])
def test_mini_bf16_attention_without_parts(n_prefix, K, monkeypatch):
    """The barrier-free kernel's attention of short prefixes (one workgroup per row tile walks every chunk): one, two
    and three rounds of chunks per wave, new positions crossing a chunk boundary, the longest prefix the mode takes."""
    from tests.parity import run_verify_parity
    monkeypatch.setenv("SSD_ATTN_WHOLE", "1")
    r = run_verify_parity("mini", steps=3, K=K, beta=0.3, atol_logits=2e-2, atol_probs=2e-2, n_prefix=n_prefix)
    assert r["path"] == 4, "attention without parts did not run"


@pytest.mark.gpu
@pytest.mark.parametrize("flight,K", [("2", 0), ("2", 7), ("4", 3), ("4", 7), ("10", 7), ("16", 0), ("18", 0), ("2", 12),
                                      ("", 1), ("", 3)])
def test_mini_bf16_operand_staging_flights(flight, K, monkeypatch):
    """The barrier-free kernel is instantiated per number of rows that it keeps in flight while it stages GEMM operands (2, 4, 6, 8, 10 for
    SSD_DF_FLIGHT=2, 4, 10, 16, 18; chosen per launch from the row count): every instantiation, those of 2 and 4 rows also with rows that
    need several flights, more than the 8 rows up to which one can be asked for, and the launch's own choice."""
    from tests.parity import run_verify_parity
    if flight:
        monkeypatch.setenv("SSD_DF_FLIGHT", flight)
    else:
        monkeypatch.delenv("SSD_DF_FLIGHT", raising=False)
    r = run_verify_parity("mini", steps=3, K=K, beta=0.3, atol_logits=2e-2, atol_probs=2e-2)
    assert r["path"] == 3, "the barrier-free persistent kernel did not run"


@pytest.mark.gpu
@pytest.mark.parametrize("d,ffn", [(96, 64), (160, 6208), (64, 2048), (32, 2080), (1120, 96)])
def test_sums_of_down_projection_partials(d, ffn):
    """The sums over the workgroups' partial results of the down projection, which are there when they are not zero and are put back to
    zero: fewer partials than blocks of them (2), one per block (64), one more, and four of a block where three are in flight; the last 64 columns with
    and without their second half.  Every third output column's partials are exact zeros.  Three layers use a buffer twice, and launches
    of 1, 2, 5, 8, 9 and 16 rows, which have it in three layouts, follow each other on one cache, as do the two sets of the other words
    (1120 columns: more than a flight's)."""
    from tests.parity import Pair, loud_weights, verify_parity_step
    shape = dict(n_layers=3, d_model=d, n_q_heads=2, n_kv_heads=1, head_dim=64, d_ffn=ffn, vocab=41, n_embed=43, dtype="bf16",
                 qkv_bias=1, rope_base=1.0e4, rms_eps=1e-6)
    w = loud_weights(shape, 87)
    for l in range(3):
        w[f"l{l}.wdown"][::3] = 0.0
    pair = Pair(None, 0, 128, max_rows=16, shape=shape, weights=w, store="bf16")
    rng = np.random.default_rng(88)
    pair.prefill(0, rng.integers(0, 43, 12))
    for s, K in enumerate((0, 1, 4, 7, 8, 15, 0, 8, 4)):
        verify_parity_step(pair, dict(beta=0.3, seed=89), K, s, rng, 2.0 ** -4, 2.0 ** -4)       # (as check_prompt's elements)
        assert pair.kv.last_forward_path() in (3, 4), "the barrier-free persistent kernel did not run"
        pair.check_rows(0, 2.0 ** -7)
    pair.check_free_stack()


@pytest.mark.gpu
@pytest.mark.parametrize("n_prefix", [12, 1540])
def test_handed_over_words_whose_value_is_zero(n_prefix):
    """Every kind of value that one workgroup hands another as a word which is not zero, being zero: embedding rows, products with a norm's gain
    and sums of squares (every other token's embedding is zero, every fifth gain), queries of a whole head, halves of the new keys and values,
    residual columns behind the output and the down projection; in launches of 1 to 16 rows on one cache, which use both sets of the words, with
    attention in one part and in two."""
    from tests.parity import Pair, loud_weights, verify_parity_step
    shape = dict(n_layers=2, d_model=96, n_q_heads=2, n_kv_heads=1, head_dim=64, d_ffn=64, vocab=41, n_embed=43, dtype="bf16",
                 qkv_bias=1, rope_base=1.0e4, rms_eps=1e-6)
    w = loud_weights(shape, 97)
    w["embed"][::2] = 0.0
    w["final_norm"][::5] = 0.0
    zero = np.r_[0:64, 128:144, 160:176, 192:224]            # of q head 0, of the keys (both dims of a rotated pair), of the values
    for l in range(2):
        w[f"l{l}.ln1"][::5] = w[f"l{l}.ln2"][::5] = 0.0
        w[f"l{l}.wqkv"][zero] = 0.0
        w[f"l{l}.bqkv"][zero] = 0.0
        w[f"l{l}.wo"][::3] = 0.0
        w[f"l{l}.wdown"][::3] = 0.0
    pair = Pair(None, 0, n_prefix + 96, max_rows=16, shape=shape, weights=w, store="bf16")
    rng = np.random.default_rng(98)
    pair.prefill(0, rng.integers(0, 43, n_prefix))
    for s, K in enumerate((0, 1, 4, 7, 8, 15, 0, 8)):
        verify_parity_step(pair, dict(beta=0.3, seed=99), K, s, rng, 2.0 ** -4, 2.0 ** -4)
        assert pair.kv.last_forward_path() in (3, 4), "the barrier-free persistent kernel did not run"
        pair.check_rows(0, 2.0 ** -7)
    pair.check_free_stack()


@pytest.mark.gpu
def test_barrier_and_barrier_free_kernels_agree(monkeypatch):
    """Same model, prefix and drafts through both persistent kernels: logits agree to rounding (they share the
    arithmetic definitions but not every summation order), decisions given equal probabilities are covered above."""
    import torch
    import synth_inputs as si
    import paper_2505_15380_amd as ssd
    wl = si.workload("mini")
    shape = si.model_shape(wl["target"])
    w = si.make_weights(shape, wl["seeds"]["target"])
    toks = si.make_prefix(shape, 0, 300, wl["seeds"]["prefix"])
    K, V = 4, shape["vocab"]
    outs = []
    for mode, whole, want in (("barrier", "0", 2), ("", "0", 3), ("", "1", 4)):
        monkeypatch.setenv("SSD_ATTN_WHOLE", whole)
        if mode:
            monkeypatch.setenv("SSD_FORWARD", mode)
        else:
            monkeypatch.delenv("SSD_FORWARD", raising=False)
        cfg = ssd.sample_config(beta=0.0, seed=3)
        sess = ssd.SSDSession(shape, w, None, None, 1, K, len(toks) + 64, cfg, cfg)
        sess.prefill(0, torch.from_numpy(toks).cuda())
        x = torch.arange(5, 5 + K, dtype=torch.int32, device="cuda").reshape(1, K)
        pd = torch.full((1, K, V), 1.0 / V, dtype=torch.float32, device="cuda")
        logits = torch.zeros((1, K + 1, V), dtype=torch.float32, device="cuda")
        ssd.ssd_verify(sess.target, sess.kv, 1, x, pd, K, cfg, 0,
                       out=dict(n_accepted=sess.n_acc, next_token=sess.next, probs=None, logits=logits))
        torch.cuda.synchronize()
        assert sess.kv.last_forward_path() == want
        outs.append(logits.cpu().numpy())
    assert all(np.isfinite(o).all() for o in outs)
    assert np.abs(outs[0] - outs[1]).max() < 2e-3 and np.abs(outs[1] - outs[2]).max() < 2e-3


@pytest.mark.gpu
def test_mini_bf16_parity_with_matched_cache_format():
    """Against the oracle whose cache holds keys/values as the bf16 pool does, what remains is the arithmetic of the
    kernels: an order of magnitude inside the 2e-2 that the exact oracle is met with (most of which is the format)."""
    from tests.parity import run_verify_parity
    r = run_verify_parity("mini", steps=6, K=4, beta=0.2, atol_logits=4e-3, atol_probs=4e-3, atol_kv=1.6e-2, store="bf16")
    assert 0 < r["dlogits"] < 4e-3
