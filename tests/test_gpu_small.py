"""GPU tests of the fp32 forward of a few rows as one launch: the bits of the launches per operator, at the edges of its items and of what it takes."""
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


SHAPES = {
    "tiny": {},
    "narrowest": dict(n_layers=1, d_model=32, n_q_heads=1, n_kv_heads=1, d_ffn=32, vocab=17, n_embed=17),              # waves without a step
    "one_head": dict(n_layers=3, d_model=224, n_q_heads=1, n_kv_heads=1, d_ffn=96, vocab=65, n_embed=65),                # waves without a step, four rounds of residual columns
    "grouped": dict(n_layers=3, d_model=192, n_q_heads=6, n_kv_heads=2, d_ffn=320, vocab=777, n_embed=800, qkv_bias=1),  # five waves for the down projection
    "widest": dict(n_layers=2, d_model=256, n_q_heads=8, n_kv_heads=8, d_ffn=512, vocab=513, n_embed=513, qkv_bias=1),
    "ten_heads": dict(n_layers=2, d_model=128, n_q_heads=8, n_kv_heads=1, d_ffn=512, vocab=513, n_embed=513, qkv_bias=1),  # to a workgroup of attention
    "group_of_3": dict(n_layers=2, d_model=256, n_q_heads=6, n_kv_heads=2, d_ffn=512, vocab=513, n_embed=513, qkv_bias=1),
    "group_of_4": dict(n_layers=2, d_model=256, n_q_heads=8, n_kv_heads=2, d_ffn=512, vocab=513, n_embed=513, qkv_bias=1),  # faster per operator
}


def _run(shape, w, lens, K, pcap, steps):
    import paper_2505_15380_amd as ssd
    B, V, cap = len(lens), shape["vocab"], max(lens) + 200
    model = ssd.Model(shape, w, cap)
    kv = ssd.KVCache(model, B, max(32, K + 1), sum(-(-(n + 200) // 16) for n in lens), 16, -(-cap // 16), pcap)
    rng, outs, paths = np.random.default_rng(3), [], []
    for b, n in enumerate(lens):
        toks = np.random.default_rng(1000 + b).integers(0, V, n + 1).astype(np.int32)
        ssd.ssd_prefill(model, kv, b, torch.from_numpy(toks).cuda())
    for s in range(steps):
        if pcap == 2:
            x, p = torch.zeros(B, dtype=torch.int32, device="cuda"), torch.zeros(B, V, device="cuda")
            ssd.ssd_draft_step(model, kv, B, ssd.sample_config(seed=4), s, 0, x, 1, p, V)
            outs += [x, p]
            if s == 1:                       # two pending tokens, one of two: the next step has a row that carries nothing
                drafts = x[:, None].contiguous()
                ssd.ssd_kv_follow(kv, B, 1, torch.tensor([b % 2 for b in range(B)], dtype=torch.int32, device="cuda"), x, drafts)
        else:
            x = torch.from_numpy(rng.integers(0, V, (B, K)).astype(np.int32)).cuda() if K else None
            pd = torch.full((B, K, V), 1.0 / V, device="cuda") if K else None
            o = ssd.ssd_verify(model, kv, B, x, pd, K, ssd.sample_config(beta=0.3, seed=3), s, want_logits=True)
            outs += [o["logits"], o["n_accepted"], o["next_token"]]
        paths.append(kv.last_forward_path())
    torch.cuda.synchronize()
    return [t.clone() for t in outs] + [kv.pool.clone()], paths, [kv.state(b) for b in range(B)], kv.free_stack()


@pytest.mark.parametrize("name,lens,K,pcap,path", [
    ("tiny", [3], 0, 1, 5), ("tiny", [64], 4, 1, 5), ("tiny", [63], 1, 1, 5), ("tiny", [500], 7, 1, 5), ("tiny", [7] * 8, 7, 1, 5),
    ("tiny", [600, 2], 12, 1, 5), ("tiny", [40] * 4, 15, 1, 5), ("tiny", [30] * 16, 0, 1, 5), ("tiny", [50, 9], 0, 2, 5),
    ("tiny", [1010], 3, 1, 1),               # two parts of attention from the third verification on
    ("tiny", [20] * 5, 12, 1, 1),            # 65 rows
    ("tiny", [20] * 17, 0, 1, 1),            # 17 sequences
    ("one_head", [40], 15, 1, 5), ("one_head", [33, 5, 70], 10, 1, 5), ("one_head", [21], 8, 1, 5),
    ("narrowest", [1], 2, 1, 5), ("narrowest", [90, 14], 0, 2, 5), ("grouped", [31], 4, 1, 5), ("grouped", [100, 5, 300], 5, 1, 5),
    ("grouped", [17, 15, 16], 0, 2, 5), ("widest", [129], 8, 1, 5), ("widest", [12] * 3, 15, 1, 5),
    ("ten_heads", [129], 8, 1, 5), ("ten_heads", [12] * 3, 15, 1, 5), ("group_of_3", [12] * 3, 15, 1, 5), ("group_of_4", [40], 4, 1, 1)])
def test_one_launch_has_the_bits_of_the_launches_per_operator(name, lens, K, pcap, path, monkeypatch):
    """Logits, draws, the cache's pool, lengths, tables and free blocks after four steps; `path`: of the last of them."""
    import paper_2505_15380_amd as ssd
    shape = dict(si.model_shape("tiny"), **SHAPES[name])
    w = ssd.upload_weights(shape, si.make_weights(shape, 150))
    got = {}
    for mode in ("", "barrier"):
        if mode:
            monkeypatch.setenv("SSD_FORWARD", mode)
        else:
            monkeypatch.delenv("SSD_FORWARD", raising=False)
        got[mode] = _run(shape, w, lens, K, pcap, 4)
    a, b = got[""], got["barrier"]
    assert a[1][-1] == path and set(b[1]) == {1}
    assert all(torch.equal(x, y) for x, y in zip(a[0], b[0]))
    assert a[2:] == b[2:]


def test_launches_of_changing_rows_leave_no_words_behind(monkeypatch):
    """Launches of one to four row tiles in turn, over a workspace of two sets of words: each zeroes what the one before left, also with fewer
    row tiles than that had.  Bits of the launches per operator after each."""
    import paper_2505_15380_amd as ssd
    shape = si.model_shape("tiny")
    w = ssd.upload_weights(shape, si.make_weights(shape, 150))
    V, got = shape["vocab"], []
    for mode in ("", "barrier"):
        if mode:
            monkeypatch.setenv("SSD_FORWARD", mode)
        model = ssd.Model(shape, w, 400)
        kv = ssd.KVCache(model, 4, 64, 4 * 25, 16)
        for b in range(4):
            toks = np.random.default_rng(1000 + b).integers(0, V, 30 + 9 * b).astype(np.int32)
            ssd.ssd_prefill(model, kv, b, torch.from_numpy(toks).cuda())
        rng, outs = np.random.default_rng(3), []
        for s, (B, K) in enumerate([(4, 15), (1, 0), (4, 11), (2, 15), (3, 4), (4, 15), (4, 15), (1, 7), (1, 7), (4, 12)]):
            x = torch.from_numpy(rng.integers(0, V, (B, K)).astype(np.int32)).cuda() if K else None
            pd = torch.full((B, K, V), 1.0 / V, device="cuda") if K else None
            o = ssd.ssd_verify(model, kv, B, x, pd, K, ssd.sample_config(beta=0.3, seed=3), s, want_logits=True)
            assert kv.last_forward_path() == (1 if mode else 5)
            outs += [o["logits"].clone(), o["next_token"].clone(), kv.pool.clone()]
        got.append(outs)
    assert all(torch.equal(a, b) for a, b in zip(*got))
