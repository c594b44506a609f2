"""GPU tests: the bits of a row depend on its sequence and its position, not on what the host knows of the lengths and not on
the other sequences of the launch (include/ssd.h, "Reproducibility")."""
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
    pkg.load_library()


def _target(shape, lens, max_rows, extra=64, seed=150):
    """A target cache with sequences of the given cached lengths; the first one's prompt does not depend on the others."""
    import paper_2505_15380_amd as ssd
    cap = max(lens) + extra
    model = ssd.Model(shape, ssd.upload_weights(shape, si.make_weights(shape, seed)), cap)
    mbps = -(-cap // 16)
    kv = ssd.KVCache(model, len(lens), max_rows, sum(-(-(n + extra) // 16) for n in lens), 16, mbps, 1)
    for b, n in enumerate(lens):
        toks = np.random.default_rng(1000 + b).integers(0, shape["vocab"], n + 1).astype(np.int32)
        ssd.ssd_prefill(model, kv, b, torch.from_numpy(toks).cuda())
    return model, kv


def _verify_logits(model, kv, B, x):
    import paper_2505_15380_amd as ssd
    K, V = x.shape[1], model.shape["vocab"]
    pd = torch.full((B, K, V), 1.0 / V, device="cuda") if K else None
    out = ssd.ssd_verify(model, kv, B, x.contiguous() if K else None, pd, K, ssd.sample_config(seed=3), 0, want_logits=True)
    torch.cuda.synchronize()
    return out["logits"].clone(), kv.last_forward_path()


@pytest.mark.parametrize("shape_name,K,cached", [
    ("mini_bf16", 7, 60),          # rows on both sides of a chunk
    ("mini_bf16", 7, 1020),
    ("mini_bf16", 7, 1514),        # the bound of a verification's attention is beyond one part, that of a step is not
    ("mini_bf16", 4, 1521),
    ("mini_bf16", 7, 1530),        # some rows are the last that attend in one part, the others go in several
    ("mini_bf16", 12, 1535),
    ("mini_bf16", 4, 2046),        # a further part begins
    ("tiny", 4, 62),
    ("tiny", 4, 1022),             # fp32: rows on both sides of the end of the first part
    ("tiny", 4, 2045)])
def test_rows_verified_together_have_the_bits_of_rows_decoded_alone(shape_name, K, cached):
    """The logits of the K + 1 rows of a verification against K + 1 autoregressive steps over the same tokens."""
    import paper_2505_15380_amd as ssd
    shape = si.model_shape(shape_name)
    model, kv = _target(shape, [cached], 256)
    x = torch.from_numpy(np.random.default_rng(7).integers(0, shape["vocab"], (1, K)).astype(np.int32)).cuda()
    pending = kv.state(0)["pending"][0]
    together, path = _verify_logits(model, kv, 1, x)
    for i, tok in enumerate([pending] + x[0].tolist()):
        ssd.ssd_kv_rollback(kv, 0, cached + i, tok)
        alone, path1 = _verify_logits(model, kv, 1, x[:, :0])
        assert (path1 in (3, 4)) == (path in (3, 4))
        assert torch.equal(alone[0, 0], together[0, i]), f"row {i}: differs by {float((alone[0, 0] - together[0, i]).abs().max())}"


@pytest.mark.parametrize("n_prefix", [1010, 1290, 1500])
def test_captured_cycle_has_the_bits_of_the_eager_one_at_long_prefixes(n_prefix):
    """A cycle is captured for lengths 256 positions ahead of today's: where the eager launches, whose bound is nearer,
    could choose another cut of the attention (prefixes between about 1265 and 1520 positions)."""
    from tests.test_gpu_cycle import make_session
    import paper_2505_15380_amd as ssd
    K, cycles = 4, 10
    a, _ = make_session("mini", K, steps=60, n_prefix=n_prefix)           # (room for the bounds of the capture)
    b, _ = make_session("mini", K, steps=60, n_prefix=n_prefix)
    a.cfg = b.cfg = ssd.sample_config(beta=0.3, seed=77)
    a.dcfg = b.dcfg = ssd.sample_config(seed=78)
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    g = a.graph_cycle()
    with torch.cuda.stream(side):
        for c in range(cycles):
            g.launch()
            b.cycle(c)
            side.synchronize()
            assert torch.equal(a.x, b.x) and torch.equal(a.pd, b.pd), c
            assert int(a.n_acc[0]) == int(b.n_acc[0]) and int(a.next[0]) == int(b.next[0]), c
            if c % 4 == 3:                                 # the eager session's bounds become exact
                n = b.kv.state(0)["len"]
                for l in range(a.kv.model.shape["n_layers"]):
                    for u, v in zip(a.kv.gather(0, l, n), b.kv.gather(0, l, n)):
                        assert np.array_equal(u, v), (c, l)
    torch.cuda.synchronize()


@pytest.mark.parametrize("shape_name,B,K,cached,others", [
    ("mini_bf16", 2, 4, 1300, (40, 1700)),     # 10 rows: the barrier-free kernel
    ("mini_bf16", 32, 1, 300, (40, 900)),      # 64 rows: one launch per operator
    ("mini128_bf16", 32, 1, 300, (40, 900)),
    ("mini128_bf16", 4, 4, 620, (40, 1700)),
    ("tiny", 2, 4, 1000, (40, 1100)),
    ("tiny", 2, 4, 1100, (40, 2100))])
def test_a_sequences_bits_do_not_depend_on_the_lengths_of_the_others(shape_name, B, K, cached, others):
    """The same first sequence in two batches of one shape, beside short sequences and beside long ones."""
    shape = si.model_shape(shape_name)
    got = []
    for n in others:
        model, kv = _target(shape, [cached] + [n] * (B - 1), 32)
        x = torch.from_numpy(np.random.default_rng(7).integers(0, shape["vocab"], (B, K)).astype(np.int32)).cuda()
        logits, path = _verify_logits(model, kv, B, x)
        got.append(logits[0])
    assert torch.equal(got[0], got[1]), f"differs by {float((got[0] - got[1]).abs().max())}"


@pytest.mark.parametrize("K", [0, 4, 7])
def test_words_in_flight_do_not_change_bits(K, monkeypatch):
    """Every instantiation of the barrier-free kernel on the same rows of width 896: one flight or several (eight rows need two
    of the 10-word ones), both halves of an operand in one matrix instruction or in two, sums of squares over 8 or 32 columns."""
    shape = si.model_shape("half_b_draft")
    shape.update(n_layers=1, vocab=300, n_embed=300)
    x = torch.from_numpy(np.random.default_rng(7).integers(0, 300, (1, K)).astype(np.int32)).cuda()
    got = []
    for flight in ("", "2", "4", "10", "16", "18"):
        if flight:
            monkeypatch.setenv("SSD_DF_FLIGHT", flight)
        else:
            monkeypatch.delenv("SSD_DF_FLIGHT", raising=False)
        logits, path = _verify_logits(*_target(shape, [70], 64), 1, x)
        assert path == 3
        got.append(logits)
    assert all(torch.equal(g, got[0]) for g in got[1:])


@pytest.mark.parametrize("B,R", [(33, 1), (40, 5), (40, 7), (64, 3)])
def test_attention_of_launches_that_leave_half_of_the_device_idle(B, R, monkeypatch):
    """Between a quarter and half of the device's compute units in workgroups of four row tiles: the launch takes two tiles x four
    key groups instead (one row tile, an odd number of them, up to twelve chunks, one chunk and fewer).  Against the vector-unit
    kernel on the same cache: both keep 16 bits and more of every operand (2^-17 relative), so the logits, of the order of 1, agree to 1e-3."""
    import paper_2505_15380_amd as ssd
    shape = si.model_shape("mini_bf16")
    rng = np.random.default_rng(5)
    lens = [int(n) for n in rng.integers(1, 760, B)]
    lens[:4] = [1, 63, 64, 759]
    x = torch.from_numpy(rng.integers(0, shape["vocab"], (B, R - 1)).astype(np.int32)).cuda()
    got = {}
    for mode in ("valu", ""):
        monkeypatch.setenv("SSD_ATTN", mode)
        model, kv = _target(shape, lens, 1024 // B)
        got[mode], path = _verify_logits(model, kv, B, x)
        assert path == 1
    assert (got["valu"] - got[""]).abs().max() < 1e-3
    assert got[""].abs().max() > 0.1


@pytest.mark.parametrize("K", [0, 1, 5])
def test_a_small_model_beside_a_large_one_on_another_stream(K):
    """The workgroups of a barrier-free launch wait for each other, so launches on two streams have to fit the device together: at width 896
    one takes 218 compute units, and a small model's 13 have room beside it.  The same steps as one after the other."""
    import paper_2505_15380_amd as ssd
    large = si.model_shape("half_b_draft")
    large.update(vocab=300, n_embed=300)
    small = dict(n_layers=4, d_model=64, n_q_heads=2, n_kv_heads=1, head_dim=64, d_ffn=64, vocab=41, n_embed=43, dtype="bf16", qkv_bias=1,
                 rope_base=1.0e4, rms_eps=1e-6)
    runs = []
    for shape in (large, small):
        model, kv = _target(shape, [70], 64, extra=400)
        x = torch.from_numpy(np.random.default_rng(7).integers(0, shape["vocab"], (1, K)).astype(np.int32)).cuda() if K else None
        pd = torch.full((1, K, shape["vocab"]), 1.0 / shape["vocab"], device="cuda") if K else None
        runs.append((model, kv, x, pd, torch.cuda.Stream(), kv.state(0)["pending"][0]))
    cfg = ssd.sample_config(beta=0.3, seed=3)
    got = []
    for beside in (False, True):
        for _, kv, _, _, stream, pending in runs:
            with torch.cuda.stream(stream):
                ssd.ssd_kv_rollback(kv, 0, 70, pending)
        torch.cuda.synchronize()
        outs = []
        for step in range(20):
            for model, kv, x, pd, stream, _ in runs:
                with torch.cuda.stream(stream):
                    outs.append(ssd.ssd_verify(model, kv, 1, x, pd, K, cfg, step, want_logits=True)["logits"])
                    assert kv.last_forward_path() in (3, 4)
                if not beside:
                    torch.cuda.synchronize()
        torch.cuda.synchronize()
        got.append(outs)
    assert all(torch.equal(a, b) for a, b in zip(*got))
