"""GPU tests of the barrier-free forward's wide form (head size 128): against the oracle at the edges of its tiles, phases and row counts, the bits of its
rows, and two such launches on two streams."""
import numpy as np
import pytest
import torch

import synth_inputs as si

pytestmark = pytest.mark.gpu

WIDE = dict(n_layers=2, d_model=1536, n_q_heads=12, n_kv_heads=2, head_dim=128, d_ffn=8960, vocab=300, n_embed=300, dtype="bf16", qkv_bias=1,
            rope_base=1.0e6, rms_eps=1e-6)


@pytest.fixture(scope="module", autouse=True)
def need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2505_15380_amd as pkg
    pkg.load_library()


def _shape(name):
    if name == "mini128":
        return si.model_shape("mini128_bf16")
    s = dict(WIDE)
    if name == "odd":            # one kv head, width of 3 x 32 (a last sum task of half a width), 301 k-tiles of the down projection: the last workgroup has one
        s.update(d_model=96, n_q_heads=3, n_kv_heads=1, d_ffn=32 * 301)
    if name == "one_layer":
        s.update(n_layers=1)
    if name == "eight_heads":    # items of the output projection two to a workgroup, and one row's operands two pieces of 512 words: half of the threads have none
        s.update(n_layers=3, n_q_heads=8, d_ffn=32 * 192)
    if name == "four_heads":     # the same with two rows
        s.update(n_layers=3, n_q_heads=4, d_ffn=32 * 200)
    return s


@pytest.mark.parametrize("name,lens,K", [
    ("mini128", [40], 0), ("mini128", [63], 1), ("mini128", [1010], 4), ("mini128", [1530], 7), ("mini128", [2040], 12),
    ("mini128", [5, 130], 5), ("mini128", [1535, 20, 300], 3), ("odd", [33], 2), ("odd", [150], 8), ("odd", [70], 15), ("odd", [1100], 3),
    ("one_layer", [20], 0), ("one_layer", [50], 7), ("one_layer", [18], 12), ("one_layer", [45], 15), ("mini128", [5116], 7),
    ("eight_heads", [40], 0), ("eight_heads", [40], 2), ("four_heads", [40], 1), ("four_heads", [30], 0)])
def test_wide_forward_against_the_oracle(name, lens, K):
    """Two verifications each, and the cached keys and values after each.  Rows 1 to 16 (sums of 8, 32 and 64 columns, both halves of an operand in one
    instruction or in two), new rows within a chunk, across chunks, across the end of the only part and into a sixth part (five are merged in one flight).  With the cache's format in the oracle
    what is left are fp32 sums and keys that round the other way, as in test_mini_bf16_parity_with_matched_cache_format, whose bounds these are."""
    from tests.parity import Pair, verify_parity_step
    shape = _shape(name)
    steps = 2
    pair = Pair(None, 881, max(lens) + steps * (K + 1) + 20, max_seqs=len(lens), max_rows=256, shape=shape, store="bf16")
    for b, n in enumerate(lens):
        pair.prefill(b, np.random.default_rng(90 + b).integers(0, shape["n_embed"], n + 1))
    rng = np.random.default_rng(12)
    for s in range(steps):
        verify_parity_step(pair, dict(beta=0.2, temperature=1.0, top_k=0, greedy=False, seed=77), K, s, rng, 4e-3, 4e-3, seqs=range(len(lens)))
        assert pair.kv.last_forward_path() == 3
        for b in range(len(lens)):
            pair.check_state(b, 1.6e-2)
        pair.check_free_stack()


@pytest.mark.parametrize("name,K,rows", [("mini128", 7, 8), ("mini128", 12, 13), ("odd", 15, 16), ("one_layer", 5, 6), ("one_layer", 15, 16)])
def test_wide_rows_of_a_prompt_with_loud_weights(name, K, rows):
    """A prompt in launches of `rows` rows, on weights with which a lost piece of a tile counts: each cached row within one step of bf16 of the oracle's."""
    from tests.parity import Pair, loud_weights
    shape = dict(_shape(name), n_layers=2)
    if name == "one_layer":
        shape.update(d_ffn=32 * 185)                       # more k-tiles than workgroups: 93 workgroups, the last with one
    pair = Pair(None, 0, 96, max_rows=rows, shape=shape, weights=loud_weights(shape, 31), store="bf16")
    pair.prefill(0, np.random.default_rng(32).integers(0, shape["n_embed"], 3 * rows + 2))
    assert pair.kv.last_forward_path() == 3
    pair.check_rows(0, 2.0 ** -7)


@pytest.mark.parametrize("name,K,cached", [("mini128", 7, 60), ("mini128", 7, 1514), ("mini128", 7, 1530), ("mini128", 12, 1535), ("mini128", 4, 2046),
                                           ("one_layer", 4, 100), ("one_layer", 15, 120), ("odd", 12, 1020), ("mini128", 7, 5116), ("mini128", 15, 6140),
                                           ("eight_heads", 7, 60), ("four_heads", 3, 60)])
def test_wide_rows_verified_together_have_the_bits_of_rows_decoded_alone(name, K, cached):
    from tests.test_gpu_row_bits import _target, _verify_logits
    import paper_2505_15380_amd as ssd
    shape = _shape(name)
    model, kv = _target(shape, [cached], 256)
    x = torch.from_numpy(np.random.default_rng(7).integers(0, shape["vocab"], (1, K)).astype(np.int32)).cuda()
    pending = kv.state(0)["pending"][0]
    together, path = _verify_logits(model, kv, 1, x)
    assert path == 3
    for i, tok in enumerate([pending] + x[0].tolist()):
        ssd.ssd_kv_rollback(kv, 0, cached + i, tok)
        alone, path = _verify_logits(model, kv, 1, x[:, :0])
        assert path == 3
        assert torch.equal(alone[0, 0], together[0, i]), f"row {i}: differs by {float((alone[0, 0] - together[0, i]).abs().max())}"


@pytest.mark.parametrize("other", ["wide", "narrow", "three"])
def test_launches_that_do_not_fit_the_device_together_are_ordered(other):
    """Two models on two streams, issued in turn without a wait in between; 204 and more workgroups each.  The same steps as one after the other.
    "three": and a small one on a third, which fits beside one of them but has to mind what that one is ordered behind."""
    from tests.test_gpu_row_bits import _target
    import paper_2505_15380_amd as ssd
    second = _shape("one_layer") if other == "wide" else dict(si.model_shape("half_b_draft"), vocab=300, n_embed=300)
    K, runs = 4, []
    for shape in [_shape("wide"), second] + [si.model_shape("tiny")] * (other == "three"):
        model, kv = _target(shape, [70], 64, extra=400)
        x = torch.from_numpy(np.random.default_rng(7).integers(0, shape["vocab"], (1, K)).astype(np.int32)).cuda()
        pd = torch.full((1, K, shape["vocab"]), 1.0 / shape["vocab"], device="cuda")
        runs.append((model, kv, x, pd, torch.cuda.Stream(), kv.state(0)["pending"][0]))
    cfg = ssd.sample_config(beta=0.3, seed=3)
    got = []
    for beside in (False, True):
        for _, kv, _, _, stream, pending in runs:
            with torch.cuda.stream(stream):
                ssd.ssd_kv_rollback(kv, 0, 70, pending)
        torch.cuda.synchronize()
        outs = []
        for step in range(12):
            for model, kv, x, pd, stream, _ in runs:
                with torch.cuda.stream(stream):
                    outs.append(ssd.ssd_verify(model, kv, 1, x, pd, K, cfg, step, want_logits=True)["logits"])
                    assert kv.last_forward_path() in (3, 4, 5)
                if not beside:
                    torch.cuda.synchronize()
        torch.cuda.synchronize()
        got.append(outs)
    assert all(torch.equal(a, b) for a, b in zip(*got))


def test_launches_of_threads_on_their_own_streams_are_ordered(monkeypatch):
    """hipStreamPerThread is one handle for a stream of each thread: two threads that issue launches of 204 and 218 workgroups on it at once.
    The same steps as one after the other."""
    import threading
    import paper_2505_15380_amd as ssd
    from paper_2505_15380_amd import binding
    from tests.test_gpu_row_bits import _target
    K, runs = 4, []
    for shape in (_shape("one_layer"), dict(si.model_shape("half_b_draft"), vocab=300, n_embed=300)):
        model, kv = _target(shape, [70], 64, extra=400)
        x = torch.from_numpy(np.random.default_rng(7).integers(0, shape["vocab"], (1, K)).astype(np.int32)).cuda()
        pd = torch.full((1, K, shape["vocab"]), 1.0 / shape["vocab"], device="cuda")
        outs = [dict(n_accepted=torch.zeros(1, dtype=torch.int32, device="cuda"), next_token=torch.zeros(1, dtype=torch.int32, device="cuda"), probs=None,
                     logits=torch.zeros(1, K + 1, shape["vocab"], device="cuda")) for _ in range(40)]
        runs.append((model, kv, x, pd, outs, kv.state(0)["pending"][0]))
    cfg, got, errors = ssd.sample_config(beta=0.3, seed=3), [], []

    def steps(run):
        try:
            model, kv, x, pd, outs, pending = run
            for s in range(40):
                if s % 20 == 0:
                    ssd.ssd_kv_rollback(kv, 0, 70, pending)
                ssd.ssd_verify(model, kv, 1, x, pd, K, cfg, s, out=outs[s])
        except Exception as e:                               # (raised again in the test's own thread)
            errors.append(e)

    for beside in (False, True):
        torch.cuda.synchronize()
        if beside:
            monkeypatch.setattr(binding, "_stream", lambda: 2)
            threads = [threading.Thread(target=steps, args=(r,)) for r in runs]
            for t in threads:
                t.start()
            for t in threads:
                t.join()
            monkeypatch.undo()
        else:
            for r in runs:
                steps(r)
        torch.cuda.synchronize()
        assert not errors, errors
        assert all(r[1].last_forward_path() in (3, 4) for r in runs)
        got.append([o["logits"].clone() for r in runs for o in r[4]])
    assert all(torch.equal(a, b) for a, b in zip(*got))


@pytest.mark.parametrize("lens,K,path", [([2040, 2060], 7, 1), ([1500, 700], 7, 3), ([3090, 20], 7, 3), ([2060], 15, 3), ([2060, 2060, 30], 4, 1),
                                         ([2060, 2060], 5, 3), ([30] * 5, 2, 1)])
def test_which_batches_of_wide_rows_are_one_launch(lens, K, path):
    """More than 12 rows of several sequences whose phases share workgroups, up to 3072 positions, and more than six tiles: one launch per operator."""
    from tests.test_gpu_row_bits import _target, _verify_logits
    shape = _shape("one_layer")
    model, kv = _target(shape, lens, 128)
    x = torch.from_numpy(np.random.default_rng(7).integers(0, shape["vocab"], (len(lens), K)).astype(np.int32)).cuda()
    assert _verify_logits(model, kv, len(lens), x)[1] == path


@pytest.mark.parametrize("busy", [False, True])
def test_launches_beside_a_stream_that_is_being_captured(busy):
    """What a stream was given before its capture may still run: a launch of another stream that does not fit beside it waits for it on the host, and, where
    that takes more than a second (`busy`), runs per operator, a captured cycle call by call.  Logits within the rounding of cached keys, decisions the same."""
    import ctypes as C
    import paper_2505_15380_amd as ssd
    from tests.test_gpu_cycle import make_session
    from tests.test_gpu_row_bits import _target
    hip = ssd.load_library()                                 # (the runtime that the library is linked with)
    K, a, b = 4, torch.cuda.Stream(), torch.cuda.Stream()
    cfg = ssd.sample_config(beta=0.3, seed=3)

    def verify(shape, model, kv):
        x = torch.from_numpy(np.random.default_rng(7).integers(0, shape["vocab"], (1, K)).astype(np.int32)).cuda()
        pd = torch.full((1, K, shape["vocab"]), 1.0 / shape["vocab"], device="cuda")
        return lambda: ssd.ssd_verify(model, kv, 1, x, pd, K, cfg, 0, want_logits=True)["logits"]

    shapes = [_shape("one_layer"), dict(si.model_shape("half_b_draft"), vocab=300, n_embed=300), si.model_shape("tiny")]
    targets = [_target(s, [70], 64) for s in shapes]
    calls = [verify(s, *t) for s, t in zip(shapes, targets)]
    one, _ = make_session("mini", 3, beta=0.3, steps=8, n_prefix=60)
    two, _ = make_session("mini", 3, beta=0.3, steps=8, n_prefix=60)
    pending = [kv.state(0)["pending"][0] for _, kv in targets]
    m = torch.randn(8192, 8192, device="cuda", dtype=torch.bfloat16)
    out = torch.empty_like(m)
    torch.mm(m, m, out=out)
    torch.cuda.synchronize()
    with torch.cuda.stream(b):
        g = one.graph_cycle()
        g.launch()
        two.cycle(0)
        ref = [f() for f in calls[1:]]
        for (_, kv), p in zip(targets[1:], pending[1:]):
            ssd.ssd_kv_rollback(kv, 0, 70, p)
    torch.cuda.synchronize()
    with torch.cuda.stream(a):
        if busy:                                             # 3 to 4 seconds of products of at least 1 ms each at the card's peak, measured first
            start, stop = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            start.record()
            for _ in range(20):
                torch.mm(m, m, out=out)
            stop.record()
            a.synchronize()
            for _ in range(min(5000, int(3500 / (start.elapsed_time(stop) / 20)))):
                torch.mm(m, m, out=out)
        calls[0]()
        assert targets[0][1].last_forward_path() == 3
    graph, held = C.c_void_p(), []
    assert hip.hipStreamBeginCapture(C.c_void_p(a.cuda_stream), 1) == 0      # (thread-local)
    try:
        with torch.cuda.stream(b):
            got = [f() for f in calls[1:]]
            held.append(targets[1][1].last_forward_path())
            for c in (1, 2):
                g.launch()
                held.append(one.kv.last_forward_path())
    finally:
        assert hip.hipStreamEndCapture(C.c_void_p(a.cuda_stream), C.byref(graph)) == 0      # (nothing broke it off)
    if graph.value:
        assert hip.hipGraphDestroy(graph) == 0
    assert held == [1 if busy else 3] * 3
    torch.cuda.synchronize()
    with torch.cuda.stream(b):
        for c in (1, 2):
            two.cycle(c)
        g.launch()
        two.cycle(3)
        assert one.kv.last_forward_path() == 3
        ssd.ssd_kv_rollback(targets[1][1], 0, 70, pending[1])
        again = calls[1]()
        assert targets[1][1].last_forward_path() == 3
        torch.cuda.synchronize()
        assert torch.equal(one.x, two.x) and int(one.n_acc[0]) == int(two.n_acc[0]) and int(one.next[0]) == int(two.next[0])
        assert one.kv.state(0) == two.kv.state(0) and one.kv_d.state(0) == two.kv_d.state(0)
        # path 1 against path 3: cached keys and values of bf16 that round the other way
        assert float((one.pd - two.pd).norm()) <= 1e-2 * float(two.pd.norm())
    assert torch.equal(again, ref[0]) and torch.equal(got[1], ref[1])        # (fp32: the same bits either way)
    assert float((got[0] - ref[0]).norm()) <= 1e-2 * float(ref[0].norm())


def test_a_stream_that_was_destroyed_is_not_asked(monkeypatch):
    """Its handle may be anything by then: launches that would not have fitted beside its last ones go on as ever."""
    import ctypes as C
    import paper_2505_15380_amd as ssd
    from paper_2505_15380_amd import binding
    from tests.test_gpu_row_bits import _target, _verify_logits
    hip = ssd.load_library()
    x = torch.zeros(1, 0, dtype=torch.int32, device="cuda")
    for shape in (_shape("one_layer"), dict(si.model_shape("half_b_draft"), vocab=300, n_embed=300)):
        model, kv = _target(shape, [70], 64)
        torch.cuda.synchronize()
        st = C.c_void_p()
        assert hip.hipStreamCreate(C.byref(st)) == 0
        with monkeypatch.context() as m:
            m.setattr(binding, "_stream", lambda: st.value)
            assert _verify_logits(model, kv, 1, x)[1] == 3
        assert hip.hipStreamDestroy(st) == 0
        assert _verify_logits(model, kv, 1, x)[1] == 3


@pytest.mark.parametrize("name", ["mini128", "one_layer", "tiny"])
def test_calls_in_a_callers_graph_run_per_operator(name, monkeypatch):
    """A graph that the caller captures may be replayed beside others, which the library does not see: head size 128 and fp32 have no launches there that wait. Several
    replays, with eager calls and waits in between, against the launches per operator of a second cache."""
    import paper_2505_15380_amd as ssd
    from tests.test_gpu_row_bits import _target
    shape = si.model_shape("tiny") if name == "tiny" else _shape(name)
    K, V, caches = 3, shape["vocab"], []
    x = torch.from_numpy(np.random.default_rng(7).integers(0, V, (1, K)).astype(np.int32)).cuda()
    pd = torch.full((1, K, V), 1.0 / V, device="cuda")
    cfg = ssd.sample_config(beta=0.3, seed=3)
    for mode in ("", "barrier"):
        if mode:
            monkeypatch.setenv("SSD_FORWARD", mode)
        model, kv = _target(shape, [70], 32, extra=200)
        out = dict(n_accepted=torch.zeros(1, dtype=torch.int32, device="cuda"), next_token=torch.zeros(1, dtype=torch.int32, device="cuda"), probs=None,
                   logits=torch.zeros(1, K + 1, V, device="cuda"))
        caches.append((model, kv, out))
    (model, kv, out), (model1, kv1, out1) = caches
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        ssd.ssd_verify(model, kv, 1, x, pd, K, cfg, 0, out=out)
        assert kv.last_forward_path() == (5 if name == "tiny" else 3)
    ssd.ssd_verify(model1, kv1, 1, x, pd, K, cfg, 0, out=out1)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        ssd.ssd_verify(model, kv, 1, x, pd, K, cfg, 1, out=out)
    assert kv.last_forward_path() == 1
    for replay in range(5):
        with torch.cuda.stream(side):
            graph.replay()
        ssd.ssd_verify(model1, kv1, 1, x, pd, K, cfg, 1, out=out1)
        torch.cuda.synchronize()
        assert int(out["next_token"][0]) == int(out1["next_token"][0]) and kv.state(0)["len"] == kv1.state(0)["len"], replay
        if name == "tiny":
            assert torch.equal(out["logits"], out1["logits"]), replay
        else:
            assert float((out["logits"] - out1["logits"]).norm()) <= 1e-2 * float(out1["logits"].norm()), replay
        if replay == 2:                                      # eager work on the captured cache between replays
            with torch.cuda.stream(side):
                ssd.ssd_verify(model, kv, 1, x, pd, K, cfg, 9, out=out)
            assert kv.last_forward_path() == (5 if name == "tiny" else 3)
            ssd.ssd_verify(model1, kv1, 1, x, pd, K, cfg, 9, out=out1)
            torch.cuda.synchronize()
