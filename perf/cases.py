"""The work that users of this package have it do, as cases that can be timed and compared.

Four kinds of pass, all through the package's public calls:

  cycle    one SSD cycle of B sequences: K draft steps, one verification, the draft caches following the decision; call by
           call as SSDSession.cycle does it, or ("graph") one replay of the captured cycle
  decode   one autoregressive step of the target for B sequences (a verification without draft tokens), with the
           distribution it drew from: the baseline that speculative decoding is compared with, and its fallback
  prefill  a prompt into a sequence's cache, in launches of up to 1024 rows as SSDSession sets them up
  accept   distributions and decisions for logits that another engine computed: ssd_warp_probs, ssd_verify_from_probs

Model shapes are those of synth_inputs.  The weights are drawn on the GPU from the case's seed, with the structure that a
trained pair of models has and unrelated random ones lack: the next token is mostly predictable from the current one (the
head's row of a token is the embedding of its predecessor in a random order of the vocabulary), target distributions are
peaked (nearly all of the mass on one token, the rest spread over the vocabulary), and the draft names the target's token
four times out of five.  So acceptance is about what the paper reports, and drawn tokens seldom hang on the last bits of a
sum, as they do where thousands of tokens are equally likely.

Cycles and decoding steps let their sequences grow; after RUN passes the requests are over and the next ones start from the
same prompts (one ssd_kv_rollback per sequence and cache)."""
import math
from types import SimpleNamespace

import torch

import paper_2505_15380_amd as ssd
import synth_inputs as si

RUN = 32                     # passes between restarts
BLOCK_TOKENS = 16
DRAFT_OF = {"tiny": "tiny_draft", "half_b": "half_b_draft", "one_half_b": "one_half_b_draft"}


def listed():
    return [
        # the fp32 shape: the smallest forward there is, five of them and their samplers; all launch latency
        dict(name="tiny_fp32_cycle_k4", kind="cycle", model="tiny", B=1, K=4, lo=64, hi=64, graph=False, beta=0.4, temperature=1.0, top_k=0),
        # one stream without speculation
        dict(name="half_b_decode", kind="decode", model="half_b", B=1, K=0, lo=1024, hi=1024, beta=0.0, temperature=1.0, top_k=0),
        # the headline: one stream, one graph replay per cycle
        dict(name="half_b_cycle_k4", kind="cycle", model="half_b", B=1, K=4, lo=1024, hi=1024, graph=True, beta=0.4, temperature=1.0, top_k=0),
        # a long utterance with top-k sampling and a longer draft
        dict(name="half_b_cycle_long_k8", kind="cycle", model="half_b", B=1, K=8, lo=4096, hi=4096, graph=True, beta=0.4, temperature=1.0, top_k=25),
        # serving: sixteen streams of any age, 112 rows per verification
        dict(name="half_b_batch16_cycle_k6", kind="cycle", model="half_b", B=16, K=6, lo=256, hi=4096, graph=False, beta=0.4, temperature=1.0, top_k=0),
        # serving at the capacity of a launch: 512 rows per verification
        dict(name="half_b_batch64_cycle_k7", kind="cycle", model="half_b", B=64, K=7, lo=128, hi=1024, graph=False, beta=0.4, temperature=1.0, top_k=0),
        # the larger target (head size 128), one stream and a batch
        dict(name="one_half_b_cycle_k4", kind="cycle", model="one_half_b", B=1, K=4, lo=1024, hi=1024, graph=False, beta=0.4, temperature=1.0, top_k=0),
        dict(name="one_half_b_batch8_cycle_k8", kind="cycle", model="one_half_b", B=8, K=8, lo=1024, hi=2048, graph=False, beta=0.4, temperature=0.8, top_k=0),
        # prompts: a short one, the longest, and a ragged one on the larger target
        dict(name="half_b_prefill_97", kind="prefill", model="half_b", n=97),
        dict(name="half_b_prefill_4096", kind="prefill", model="half_b", n=4096),
        dict(name="one_half_b_prefill_1501", kind="prefill", model="one_half_b", n=1501),
        # the acceptance step for sixteen streams whose logits come from elsewhere
        dict(name="accept_b16_k6", kind="accept", B=16, K=6, V=6564, beta=0.4, temperature=0.8, top_k=25),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _sampling(rng):
    return dict(beta=rng.choice([0.0, 0.2, 0.4]), temperature=rng.choice([0.8, 1.0]), top_k=rng.choice([0, 0, 25, 50]))


def draw(rng):
    kind = rng.choice(["cycle", "cycle", "cycle", "decode", "prefill", "prefill", "accept"])
    if kind == "accept":
        return dict(kind=kind, B=_log_int(rng, 1, 64), K=rng.randint(1, 12), V=_log_int(rng, 512, 6564), **_sampling(rng))
    if kind == "prefill":
        model = rng.choice(["half_b", "half_b", "one_half_b"])
        return dict(kind=kind, model=model, n=_log_int(rng, 16, 4096 if model == "half_b" else 1501))
    model = rng.choice(["tiny", "half_b", "half_b", "half_b", "one_half_b", "one_half_b"])
    B = _log_int(rng, 1, {"tiny": 8, "half_b": 64, "one_half_b": 16}[model])
    K = 0 if kind == "decode" else rng.randint(1, 12)
    hi = _log_int(rng, 64, 512 if model == "tiny" else 4096 if B <= 16 else 1024)
    lo = hi if B == 1 else max(16, hi // rng.choice([2, 4, 16]))
    case = dict(kind=kind, model=model, B=B, K=K, lo=lo, hi=hi, **_sampling(rng))
    if kind == "cycle":                     # a cycle can be captured where both models run the persistent kernel
        case["graph"] = model == "half_b" and B * (K + 1) <= 16 and 2 * B <= 16 and rng.random() < 0.7
    return case


def _successors(V, gen):
    """succ[t]: the token that follows t.  One cycle through the vocabulary in random order."""
    order = torch.randperm(V, generator=gen, device="cuda")
    succ = torch.empty_like(order)
    succ[order] = order.roll(-1)
    return succ


def _model(shape, succ, gen, max_positions):
    """A model whose likely continuation of token t is succ[t]."""
    store = torch.bfloat16 if shape["dtype"] == "bf16" else torch.float32
    d, hd, nq, nkv, ffn, V = (shape[k] for k in ("d_model", "head_dim", "n_q_heads", "n_kv_heads", "d_ffn", "vocab"))

    def normal(*size, dtype=torch.float32):
        return torch.randn(*size, device="cuda", dtype=dtype, generator=gen)

    def mat(o, i):
        return normal(o, i, dtype=store).mul_(0.02 * math.sqrt(896 / d))       # 0.02 at the 0.5B shape's width

    def gain(n):
        return 1.0 + 0.1 * normal(n)

    embed = normal(shape["n_embed"], d, dtype=store)
    pred = torch.empty_like(succ)
    pred[succ] = torch.arange(V, device="cuda")
    # logits: about N(0, s^2 d), the predicted token 0.7 s d above them
    s = (math.log(V) + 10.0) / (0.7 * d)
    w = {"embed": embed, "final_norm": gain(d), "head": (embed[pred] * s).contiguous()}
    for l in range(shape["n_layers"]):
        w[f"l{l}.ln1"], w[f"l{l}.ln2"] = gain(d), gain(d)
        w[f"l{l}.wqkv"] = mat((nq + 2 * nkv) * hd, d)
        w[f"l{l}.bqkv"] = 0.02 * normal((nq + 2 * nkv) * hd) if shape["qkv_bias"] else None
        w[f"l{l}.wo"], w[f"l{l}.wgate"], w[f"l{l}.wup"], w[f"l{l}.wdown"] = mat(d, nq * hd), mat(ffn, d), mat(ffn, d), mat(d, ffn)
    return ssd.Model(shape, w, max_positions)


def _prompt(shape, n, gen):
    """A quarter text ids (where the shape has any), then speech ids."""
    V, E = shape["vocab"], shape["n_embed"]
    text = n // 4 if E > V else 0
    return torch.cat([torch.randint(V, E, (text,), device="cuda", generator=gen, dtype=torch.int32) if text else
                      torch.empty(0, device="cuda", dtype=torch.int32),
                      torch.randint(0, V, (n - text,), device="cuda", generator=gen, dtype=torch.int32)])


def _lengths(case):
    """Ragged prompt lengths, spread over lo .. hi."""
    return [case["lo"] + int((case["hi"] - case["lo"]) * ((b + 1) * 0.6180339887 % 1.0)) for b in range(case["B"])]


_STREAM = None


def _stream():
    """The stream of the captured cycles: HIP cannot capture the default one, and a program has one such stream for all
    its caches, since the persistent kernels of two streams would wait for each other's compute units."""
    global _STREAM
    if _STREAM is None:
        _STREAM = torch.cuda.Stream()
    return _STREAM


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    st = SimpleNamespace(kind=case["kind"], at=0)
    if st.kind == "accept":
        B, K, V = case["B"], case["K"], case["V"]
        likely = torch.randint(0, V, (B, K + 1), device="cuda", generator=gen)
        drafted = torch.where(torch.rand(B, K, device="cuda", generator=gen) < 0.2,
                              torch.randint(0, V, (B, K), device="cuda", generator=gen), likely[:, :K])

        def logits(top, rows):
            x = torch.randn(B * rows, V, device="cuda", generator=gen)
            return x.scatter_add_(1, top.reshape(-1, 1), torch.full((B * rows, 1), math.log(V) + 10.0, device="cuda"))

        st.cfg = ssd.sample_config(beta=case["beta"], temperature=case["temperature"], top_k=case["top_k"])
        st.logits = logits(likely, K + 1)
        st.pd = ssd.ssd_warp_probs(logits(drafted, K), st.cfg).view(B, K, V)
        st.x = drafted.to(torch.int32).contiguous()
        st.u = torch.randint(0, 1 << 24, (B, K + 1), device="cuda", generator=gen).float() / (1 << 24)
        st.beta, st.shape = case["beta"], (B, K + 1, V)
        return st
    shape = si.model_shape(case["model"])
    V = shape["vocab"]
    succ = _successors(V, gen)
    if st.kind == "prefill":
        n = case["n"]
        st.target = _model(shape, succ, gen, n + 64)
        st.kv = ssd.KVCache(st.target, 1, 1024, -(-(n + 64) // BLOCK_TOKENS), BLOCK_TOKENS)
        st.tokens = _prompt(shape, n + 1, gen)             # the last token stays pending: n positions are written
        return st
    B, K = case["B"], case["K"]
    lens = _lengths(case)
    grow = (RUN + 2) * (K + 1)
    max_pos = max(lens) + grow + BLOCK_TOKENS
    blocks = sum(-(-(n + grow) // BLOCK_TOKENS) + 1 for n in lens)
    st.target = _model(shape, succ, gen, max_pos)
    st.kv = ssd.KVCache(st.target, B, max(K + 1, 1024 // B), blocks, BLOCK_TOKENS)
    st.draft = None
    if K:
        dshape = si.model_shape(DRAFT_OF[case["model"]])
        wrong = torch.nonzero(torch.rand(V, device="cuda", generator=gen) < 0.2).flatten()
        dsucc = succ.clone()
        dsucc[wrong] = succ[wrong].roll(1)
        st.draft = _model(dshape, dsucc, gen, max_pos)
        st.kv_d = ssd.KVCache(st.draft, B, max(2, 1024 // B), blocks, BLOCK_TOKENS, pending_cap=2)
    prompts = [_prompt(shape, n + 1, gen) for n in lens]
    st.start = []
    for b, tokens in enumerate(prompts):
        ssd.ssd_prefill(st.target, st.kv, b, tokens)
        if K:
            ssd.ssd_prefill(st.draft, st.kv_d, b, tokens)
        st.start.append((lens[b], int(tokens[-1])))
    st.B, st.K, st.V = B, K, V
    sampling = dict(temperature=case["temperature"], top_k=case["top_k"])
    st.cfg = ssd.sample_config(beta=case["beta"], seed=seed, **sampling)
    st.dcfg = ssd.sample_config(seed=seed + 1, **sampling)
    st.out = dict(n_accepted=torch.zeros(B, dtype=torch.int32, device="cuda"), next_token=torch.zeros(B, dtype=torch.int32, device="cuda"),
                  probs=None if K else torch.zeros(B, 1, V, device="cuda"), logits=None)
    st.graph = None
    if K:
        st.x = torch.zeros(B, K, dtype=torch.int32, device="cuda")
        st.pd = torch.zeros(B, K, V, device="cuda")
        if case["graph"]:
            st.stream = _stream()
            torch.cuda.synchronize()
            with torch.cuda.stream(st.stream):
                st.graph = ssd.Cycle(st.target, st.kv, st.draft, st.kv_d, B, K, st.cfg, st.dcfg, st.x, st.pd,
                                     st.out["n_accepted"], st.out["next_token"])
    return st


def _restart(st):
    for b, (n, pending) in enumerate(st.start):
        ssd.ssd_kv_rollback(st.kv, b, n, pending)
        if st.K:
            ssd.ssd_kv_rollback(st.kv_d, b, n, pending)


def _one_cycle(st):
    B, K, V = st.B, st.K, st.V
    if st.at and st.at % RUN == 0:
        _restart(st)
    if st.graph is not None:
        st.graph.launch()
    else:
        for i in range(K):
            ssd.ssd_draft_step(st.draft, st.kv_d, B, st.dcfg, st.at, i, st.x[:, i], K, st.pd[:, i], K * V)
        ssd.ssd_verify(st.target, st.kv, B, st.x, st.pd, K, st.cfg, st.at, out=st.out)
        ssd.ssd_kv_follow(st.kv_d, B, K, st.out["n_accepted"], st.out["next_token"], st.x)
    st.at += 1


def run(st):
    if st.kind == "accept":
        pt = ssd.ssd_warp_probs(st.logits, st.cfg)
        n, token, flags = ssd.ssd_verify_from_probs(pt.view(st.shape), st.pd, st.x, st.u, st.beta)
        return dict(probs=pt, n_accepted=n, next_token=token, flags=flags)
    if st.kind == "prefill":
        ssd.ssd_prefill(st.target, st.kv, 0, st.tokens)
        return dict(cache=st.kv.pool)
    if st.kind == "decode":
        if st.at and st.at % RUN == 0:
            _restart(st)
        ssd.ssd_verify(st.target, st.kv, st.B, None, None, 0, st.cfg, st.at, out=st.out)
        st.at += 1
        return dict(next_token=st.out["next_token"], probs=st.out["probs"], cache=st.kv.pool)
    if st.graph is not None:
        with torch.cuda.stream(st.stream):
            _one_cycle(st)
    else:
        _one_cycle(st)
    return dict(drafted=st.x, draft_probs=st.pd, n_accepted=st.out["n_accepted"], next_token=st.out["next_token"],
                cache=st.kv.pool, draft_cache=st.kv_d.pool)


def _forward_work(shape, rows, rows_head, cached, attended):
    """(bytes, flops) of one forward: weights once, embedding rows, `cached` positions read, `rows` written, logits rows;
    `attended`: sum over the rows of the positions that each attends to."""
    es = 2 if shape["dtype"] == "bf16" else 4
    d, hd, nq, nkv, ffn, L, V = (shape[k] for k in ("d_model", "head_dim", "n_q_heads", "n_kv_heads", "d_ffn", "n_layers", "vocab"))
    per_layer = d * (nq + 2 * nkv) * hd + nq * hd * d + 3 * d * ffn
    head = V * d if rows_head else 0
    kv = 2 * nkv * hd * es * L
    return (L * per_layer + head) * es + rows * d * es + (cached + rows) * kv + rows_head * V * 4, \
        2 * rows * L * per_layer + 2 * rows_head * head + 4 * nq * hd * attended * L


def work(case):
    if case["kind"] == "accept":
        rows = case["B"] * (2 * case["K"] + 1)
        return {"bytes": 4 * case["V"] * (rows + case["B"] * (case["K"] + 1)), "flops": 8 * case["V"] * rows}
    shape = si.model_shape(case["model"])
    if case["kind"] == "prefill":
        n = case["n"]
        b, f = _forward_work(shape, n, 0, 0, n * (n + 1) // 2)
        return {"bytes": b, "flops": f}
    B, K = case["B"], case["K"]
    L = (case["lo"] + case["hi"]) // 2 + RUN // 2
    b, f = _forward_work(shape, B * (K + 1), B * (K + 1), B * L, B * (K + 1) * L)
    if K:
        db, df = _forward_work(si.model_shape(DRAFT_OF[case["model"]]), B, B, B * L, B * L)
        b, f = b + db, f + K * df              # the draft's weights once, its operations for every step
    return {"bytes": b, "flops": f}


def tolerance(case):
    if case["kind"] == "accept" or case["model"] == "tiny":
        return {"rel": 1e-5, "max": 4e-4}      # fp32 sums in another order
    return {"rel": 1e-2, "max": 0.1}           # bf16 storage: cached keys and values round either way
