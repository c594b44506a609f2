"""Prompts in launches of more than 1024 rows: every tile that such launches pick, and which launches there are."""
import ctypes as C

import numpy as np
import pytest
import torch

import synth_inputs as si

from tests.test_gpu_parity import check_prompt

QKV, O, GATE_UP, DOWN = 0, 2, 3, 4
BLOCK, TILE, TILE_DEEP = 1, 2, 3
# (query heads, kv heads, head size, width, ffn, rows): the tiles of QKV, output projection, gate / up and down; does down add the residual itself?
SIZES = [((9, 1, 64, 1056, 96, 1025), ((TILE, 4, 6), (TILE, 4, 8), (TILE, 8, 12), (TILE, 4, 8)), True),
         ((9, 1, 64, 32, 608, 1025), ((TILE, 4, 6), (TILE_DEEP, 4, 4), (TILE, 12, 8), (TILE_DEEP, 4, 4)), True),
         ((9, 1, 64, 32, 1056, 1025), ((TILE, 4, 6), (TILE_DEEP, 4, 4), (TILE, 12, 8), (TILE, 8, 10)), False),
         ((12, 12, 64, 2080, 96, 1025), ((TILE, 8, 6), (TILE, 8, 7), (TILE, 8, 10), (TILE, 4, 8)), True),
         ((14, 2, 64, 672, 1056, 1537), ((BLOCK, 4, 8), (TILE_DEEP, 4, 6), (TILE, 8, 12), (TILE_DEEP, 4, 6)), True),
         ((9, 1, 64, 32, 4896, 2049), ((TILE, 4, 6), (TILE_DEEP, 4, 4), (TILE, 12, 8), (TILE, 8, 7)), False),
         ((24, 8, 64, 2080, 1056, 1153), ((TILE, 8, 8), (TILE, 8, 6), (TILE, 8, 10), (TILE, 8, 7)), True),
         ((40, 8, 64, 544, 4896, 1153), ((TILE, 8, 10), (TILE_DEEP, 4, 4), (TILE, 8, 12), (TILE, 8, 12)), False),
         ((9, 1, 64, 544, 4896, 1025), ((TILE, 4, 6), (TILE_DEEP, 4, 4), (TILE, 12, 8), (TILE, 12, 8)), False),
         ((12, 12, 64, 672, 96, 3073), ((TILE, 16, 8), (TILE, 8, 7), (TILE, 8, 12), (TILE, 4, 8)), True),
         ((9, 1, 64, 1600, 4896, 1025), ((TILE, 4, 6), (TILE, 4, 8), (TILE, 8, 12), (TILE, 8, 8)), False),
         ((9, 1, 64, 1600, 4896, 1153), ((TILE, 4, 6), (TILE, 4, 8), (TILE, 8, 12), (TILE, 8, 6)), True),
         ((12, 2, 128, 96, 96, 1501), ((TILE, 4, 6), (TILE_DEEP, 4, 4), (TILE, 12, 8), (TILE, 4, 8)), True)]


def _shape(nq, nkv, hd, d, ffn):
    return dict(n_layers=2, d_model=d, n_q_heads=nq, n_kv_heads=nkv, head_dim=hd, d_ffn=ffn, vocab=41, n_embed=43, dtype="bf16",
                qkv_bias=1, rope_base=1.0e4, rms_eps=1e-6)


def _gemms(nq, nkv, hd, d, ffn):
    return (QKV, (nq + 2 * nkv) * hd, d), (O, d, nq * hd), (GATE_UP, ffn, d), (DOWN, d, ffn)


@pytest.fixture(scope="module")
def lib():
    import paper_2505_15380_amd as pkg
    return pkg.load_library()


@pytest.mark.parametrize("size,tiles,unsplit", SIZES)
def test_sizes_reach_the_tiles_they_name(lib, size, tiles, unsplit):
    plan = (C.c_int * 4)()
    for (kind, n, k), want in zip(_gemms(*size[:5]), tiles):
        assert lib.ssd_prompt_gemm_plan(kind, size[5], n, k, 256, plan, None, 0) > 0
        assert tuple(plan[:3]) == want, kind
    assert (plan[3] == 0) == unsplit


def test_blocks_of_a_prompts_launch_cover_the_output_once(lib):
    plan, blocks = (C.c_int * 4)(), (C.c_int * (3 * 65536))()
    for rows in (1, 1024, 1025, 1501, 2048, 2049, 2500, 4095, 4096):
        for n, k in ((896, 896), (1152, 896), (2048, 1536), (4864, 896), (8960, 1536), (896, 4864), (1536, 8960), (352, 64), (96, 32), (96, 8960), (352, 8960)):
            for kind in (QKV, O, GATE_UP, DOWN):
                for cus in (256, 64):
                    wgs = lib.ssd_prompt_gemm_plan(kind, rows, n, k, cus, plan, blocks, 65536)
                    assert 0 < wgs <= 65536
                    _, rt, ct, slices = plan
                    slices = slices or 1
                    assert slices * rows <= 16 * 1024 and slices <= 8      # (the partials' room)
                    got = sorted(tuple(blocks[3 * w:3 * w + 3]) for w in range(wgs) if blocks[3 * w] >= 0)
                    tiles = -(-n // 16) * (2 if kind == GATE_UP else 1)
                    assert got == sorted((c, r, s) for s in range(slices) for c in range(-(-tiles // ct)) for r in range(-(-rows // (16 * rt))))
    for rows, slices in ((1025, 8), (2048, 8), (2049, 4), (4096, 4)):     # sizes that would rather have eight where eight do not fit
        assert lib.ssd_prompt_gemm_plan(DOWN, rows, 96, 8960, 256, plan, None, 0) > 0 and plan[3] == slices
    assert lib.ssd_prompt_gemm_plan(QKV, 4097, 32, 32, 256, plan, None, 0) == -1 and lib.ssd_prompt_gemm_plan(5, 16, 32, 32, 256, plan, None, 0) == -1
    assert lib.ssd_prompt_gemm_plan(QKV, 16, 32, 32, 256, None, None, 0) == -1 and lib.ssd_prompt_gemm_plan(QKV, 16, 32, 32, 256, plan, None, 1) == -1


@pytest.mark.gpu
@pytest.mark.parametrize("size", [s[0] for s in SIZES])
def test_each_tile_against_the_oracle(size):
    """Last row tiles of one row and ragged ones, ragged last column blocks, k ranges of one k-tile and of more than the buffers hold, k-slices; sums of squares that
    the down projection leaves to the next layer."""
    check_prompt(_shape(*size[:5]), size[5], 85 + size[5] % 7)


@pytest.mark.gpu
@pytest.mark.parametrize("nq,rows,launches", [(9, 4096, 1), (9, 4181, 2), (8, 1057, 2)])
def test_which_launches_a_prompt_takes(nq, rows, launches):
    """Up to 4096 rows a launch; the rest attends to the cached ones.  Eight query heads would need partials: 1024 rows a launch."""
    import paper_2505_15380_amd as ssd
    ssd.ssd_profile_begin("qkv")
    try:
        check_prompt(_shape(nq, 1, 64, 64, 96), rows, 21)
    finally:
        _, count = ssd.ssd_profile_end()
    assert count == 2 * launches             # (two layers)


@pytest.mark.gpu
@pytest.mark.parametrize("nq,nkv,hd,seqs,rows,positions,launches", [(2, 1, 64, 4, 16, 150, 3), (9, 1, 64, 4, 16, 128, 2), (4, 2, 128, 16, 64, 1030, 2),
                                                                     (9, 9, 64, 3, 300, 905, 2), (2, 2, 32, 16, 2, 70, 3), (12, 12, 64, 8, 128, 1025, 2)])
def test_prompts_into_caches_of_several_sequences(nq, nkv, hd, seqs, rows, positions, launches):
    """A prompt takes launches of max_seqs * max_rows rows, as many as the buffers have room for, whatever the heads: also of a sequence that is not the first,
    over a cache that others have blocks in.  Against the oracle with the cache's format, as check_prompt."""
    import paper_2505_15380_amd as ssd
    from tests.parity import Pair, loud_weights
    shape = _shape(nq, nkv, hd, 64, 96)
    pair = Pair(None, 0, positions + 16, max_seqs=seqs, max_rows=rows, n_blocks=2 * (positions // 16 + 2), shape=shape, weights=loud_weights(shape, 23), store="bf16")
    pair.prefill(0, np.random.default_rng(24).integers(0, 43, 40))
    ssd.ssd_profile_begin("qkv")
    try:
        pair.prefill(seqs - 1, np.random.default_rng(25).integers(0, 43, positions + 1))
    finally:
        _, count = ssd.ssd_profile_end()
    # (a last launch of at most 16 rows that is one for all operators has no projections of its own)
    assert count in (2 * launches, 2 * (launches - 1)) and (count == 2 * launches or (positions - 1) % (seqs * rows) < 16)
    for seq in (0, seqs - 1):
        pair.check_rows(seq, 2.0 ** -7)
        pair.check_state(seq, 2.0 ** -4)
    pair.check_free_stack()


@pytest.mark.gpu
def test_fp32_prompts_have_the_same_bits_in_any_launches():
    import paper_2505_15380_amd as ssd
    shape = si.model_shape("tiny")
    w = ssd.upload_weights(shape, si.make_weights(shape, 150))
    toks = torch.from_numpy(np.random.default_rng(26).integers(0, shape["vocab"], 301).astype(np.int32)).cuda()
    got = []
    for seqs, rows in ((1, 300), (1, 16), (2, 9), (16, 64), (64, 1)):
        model = ssd.Model(shape, w, 320)
        kv = ssd.KVCache(model, seqs, rows, 20, 16)
        ssd.ssd_prefill(model, kv, 0, toks)
        torch.cuda.synchronize()
        got.append([kv.gather(0, l, 300) for l in range(shape["n_layers"])])
    assert all(np.array_equal(a[l][i], got[0][l][i]) for a in got for l in range(shape["n_layers"]) for i in (0, 1))


@pytest.mark.gpu
@pytest.mark.parametrize("nq,nkv,hd,rows,positions", [(16, 1, 64, 1024, 3301), (14, 2, 64, 1024, 1501), (12, 2, 128, 1024, 1501), (12, 2, 128, 500, 1499)])
def test_prompt_attention_where_later_scores_exceed_the_first(nq, nkv, hd, rows, positions):
    """Scores of spread 10, so that the weights' reference moves after a row's first chunk, in the forms of long prompts: eight tiles by two key groups (831
    workgroups of four tiles), four by two on head sizes 64 and 128, and on 128 a last launch of 499 rows over 24 chunks.  Against the oracle with the cache's format,
    in the 2-norm: 64 elements a key and one in 4000 a step of bf16 off, which moves 1.7 % of the rows by about 3 %, 4e-3; twice that and the format's own 2^-9."""
    from tests.parity import Pair
    shape = dict(n_layers=2, d_model=128, n_q_heads=nq, n_kv_heads=nkv, head_dim=hd, d_ffn=64, vocab=61, n_embed=61, dtype="bf16",
                 qkv_bias=0, rope_base=1.0e4, rms_eps=1e-6)
    w = si.make_weights(shape, 91)
    for l in range(2):
        w[f"l{l}.wqkv"][:(nq + nkv) * hd] *= 14.0 * (64 / hd) ** 0.25
        w[f"l{l}.wqkv"][(nq + nkv) * hd:] *= 4.0
        w[f"l{l}.wo"] *= 2.0
        for n in ("wqkv", "wo"):
            w[f"l{l}.{n}"] = torch.from_numpy(w[f"l{l}.{n}"].astype(np.float32)).bfloat16().float().numpy()
    pair = Pair(None, 0, positions + 64, max_rows=rows, shape=shape, weights=w, store="bf16")
    pair.prefill(0, np.random.default_rng(92).integers(0, 61, positions + 1))
    assert pair.kv.last_forward_path() == 1
    oc = pair.ocache[0]
    q = oc.k[0, :64, 0]
    assert np.std(q @ oc.k[0, :positions, 0].T) / hd ** 0.5 > 5.0      # (keys stand in for queries: the same distribution)
    for l in range(2):
        k, v = pair.kv.gather(0, l, oc.length)
        for got, ref in ((k, oc.k[l, :oc.length]), (v, oc.v[l, :oc.length])):
            assert np.linalg.norm(got - ref) <= 1e-2 * np.linalg.norm(ref)
