"""Which kernel and tile a bf16 forward with one launch per operator picks on 256 compute units: the sizes of the GPU tests that mean to
reach each of them do.  CPU only."""
import ctypes as C
import os

import pytest

QKV, O, GATE_UP, DOWN, HEAD = 0, 2, 3, 4, 5
KWAVE, BLOCK, TILE, TILE_DEEP = range(4)


@pytest.fixture(scope="module")
def lib():
    import paper_2505_15380_amd as pkg
    if not os.path.exists(pkg.library_path()):
        import __graft_entry__ as g
        g.build()
    return pkg.load_library()


@pytest.mark.parametrize("kind,rows,n,k,want", [
    # test_norm_between_the_projections_of_a_prompt
    (O, 65, 32, 128, (KWAVE, 1, 2)), (O, 81, 2112, 128, (KWAVE, 2, 2)), (O, 513, 1056, 128, (KWAVE, 3, 4)), (O, 961, 1056, 128, (TILE_DEEP, 4, 6)),
    (O, 1009, 1600, 128, (TILE_DEEP, 4, 8)), (O, 769, 2464, 128, (TILE, 4, 4)), (O, 961, 2080, 128, (TILE, 4, 6)), (O, 961, 3104, 128, (TILE, 4, 8)),
    # test_gate_up_and_down_at_each_tile_of_many_rows
    (GATE_UP, 65, 96, 32, (BLOCK, 4, 8)), (GATE_UP, 71, 8992, 64, (BLOCK, 5, 6)), (GATE_UP, 97, 8992, 96, (BLOCK, 7, 6)),
    (GATE_UP, 250, 4896, 64, (BLOCK, 4, 10)), (GATE_UP, 257, 8992, 32, (TILE, 4, 8)), (GATE_UP, 321, 4896, 96, (TILE, 8, 8)),
    (GATE_UP, 250, 8992, 32, (TILE, 8, 10)), (GATE_UP, 513, 4896, 64, (TILE, 8, 12)), (GATE_UP, 449, 8992, 64, (TILE, 16, 10)),
    (DOWN, 97, 96, 8992, (BLOCK, 4, 4)), (DOWN, 65, 1056, 2016, (BLOCK, 4, 8)), (DOWN, 449, 1056, 2016, (BLOCK, 8, 7)),
    (DOWN, 897, 3616, 96, (TILE, 8, 8)), (DOWN, 961, 4128, 96, (TILE, 16, 6)),
    # test_head_of_many_rows
    (HEAD, 776, 6564, 64, (TILE, 16, 8)),
    # test_qkv_projection_of_more_than_512_rows
    (QKV, 513, 256, 64, (BLOCK, 4, 4)), (QKV, 1009, 1344, 64, (BLOCK, 4, 8)), (QKV, 640, 896, 64, (BLOCK, 4, 4)), (QKV, 1024, 1408, 64, (BLOCK, 4, 8))])
def test_gemm_sizes_of_the_tests_reach_the_tiles_they_name(lib, kind, rows, n, k, want):
    plan = (C.c_int * 4)()
    assert lib.ssd_gemm_plan(kind, rows, n, k, 256, plan) == 0
    assert tuple(plan[:3]) == want


def test_every_gemm_size_has_a_plan(lib):
    """Over rows, widths and depths: the tiles cover the output, the slices the k range, and kinds that are not GEMMs are refused."""
    plan = (C.c_int * 4)()
    for kind in (QKV, O, GATE_UP, DOWN, HEAD):
        for rows in (1, 16, 17, 64, 65, 512, 513, 1024):
            for n in (32, 96, 896, 1536, 6564, 8960):
                for k in (32, 96, 896, 8960):
                    for cus in (1, 64, 256):
                        assert lib.ssd_gemm_plan(kind, rows, n, k, cus, plan) == 0
                        assert plan[1] > 0 and plan[2] > 0 and 1 <= plan[3] <= (8 if kind == DOWN else 1)
    assert lib.ssd_gemm_plan(1, 16, 32, 32, 256, plan) == -1 and lib.ssd_gemm_plan(QKV, 16, 32, 48, 256, plan) == -1
    assert lib.ssd_gemm_plan(QKV, 1025, 32, 32, 256, plan) == -1


@pytest.mark.parametrize("kind", [QKV, O, GATE_UP, DOWN, HEAD])
def test_placement_of_blocks_on_the_xcds(lib, kind):
    """Every block of the output goes to exactly one workgroup, and what the XCDs' caches fetch (a row block's activations, four bytes an input,
    by every XCD that has a block of those rows; a column block's weights, two bytes) is never more than where each XCD takes a contiguous run of
    the order (slice, column block, row block), nor are its workgroups."""
    plan, blocks = (C.c_int * 4)(), (C.c_int * (3 * 65536))()

    def fetched(of_xcd, rt, ct):
        return sum(64 * rt * len({(s, r) for _, r, s in b}) + 32 * ct * len({(s, c) for c, _, s in b}) for b in of_xcd)

    for rows in (1, 24, 65, 97, 200, 369, 477, 512, 600, 960, 1024):
        for n, k in ((896, 896), (1152, 896), (2048, 1536), (4864, 896), (8960, 1536), (896, 4864), (1536, 8960), (6564, 896), (352, 64), (96, 32)):
            for cus in (256, 64, 1):
                assert lib.ssd_gemm_plan(kind, rows, n, k, cus, plan) == 0
                _, rt, ct, slices = plan
                wgs = lib.ssd_gemm_blocks(kind, rows, n, k, cus, blocks, 65536)
                assert 0 < wgs <= 65536 and wgs % 8 == 0
                of_xcd = [[], [], [], [], [], [], [], []]
                for w in range(wgs):
                    if blocks[3 * w] >= 0:
                        of_xcd[w % 8].append(tuple(blocks[3 * w:3 * w + 3]))
                tiles = -(-n // 16) * (2 if kind == GATE_UP else 1)
                n_col, n_row = -(-tiles // ct), -(-rows // (16 * rt))
                want = [(c, r, s) for s in range(slices) for c in range(n_col) for r in range(n_row)]
                assert sorted(b for x in of_xcd for b in x) == sorted(want)
                run = -(-len(want) // 8)
                assert fetched(of_xcd, rt, ct) <= fetched([want[x * run:(x + 1) * run] for x in range(8)], rt, ct), (rows, n, k, cus, tuple(plan))
                assert max(map(len, of_xcd)) <= run
    assert lib.ssd_gemm_blocks(1, 16, 32, 32, 256, blocks, 1) == -1 and lib.ssd_gemm_blocks(QKV, 16, 32, 32, 256, None, 1) == -1
    assert lib.ssd_gemm_blocks(QKV, 16, 32, 32, 256, None, 0) > 0


@pytest.mark.parametrize("hd,nq,nkv,seqs,rows,positions,want", [
    # test_prompt_attention_where_later_scores_exceed_the_first
    (64, 10, 2, 1, 1023, 1023, (4, 2, 16)), (64, 10, 2, 1, 1023, 2046, (4, 4, 32)), (64, 10, 2, 1, 1023, 3069, (4, 4, 48)), (64, 4, 2, 1, 1024, 1024, (2, 4, 8)),
    (64, 4, 2, 1, 1024, 3072, (2, 4, 24)), (64, 7, 1, 1, 560, 3920, (4, 2, 16)), (64, 7, 1, 1, 560, 4480, (4, 4, 20)),
    # batches
    (64, 14, 2, 16, 7, 0, (4, 2, 8)), (64, 14, 2, 64, 8, 0, (2, 4, 64)), (128, 12, 2, 8, 9, 0, (4, 2, 4))])
def test_attention_sizes_of_the_tests_reach_the_forms_they_name(lib, hd, nq, nkv, seqs, rows, positions, want):
    plan = (C.c_int * 3)()
    assert lib.ssd_attention_plan(hd, nq, nkv, seqs, rows, positions, 256, plan) == 0
    assert tuple(plan) == want


def test_parts_of_attention_are_whole_rounds_of_the_key_groups(lib):
    """Over launches of every shape a sequence may have: a part's chunks are a multiple of the key groups that walk them in turn, and together
    with the row tiles they make eight or sixteen waves."""
    plan = (C.c_int * 3)()
    forms = set()
    for hd in (64, 128):
        for nq, nkv in ((1, 1), (2, 1), (7, 1), (14, 2), (12, 2), (8, 8), (32, 4)):
            for seqs in (1, 2, 7, 16, 64):
                for rows in (1, 8, 17, 100, 256, 290, 560, 1024):
                    for positions in (0,) + ((rows, rows + 1000, rows + 4100, rows + 12000) if seqs == 1 else ()):
                        if rows * seqs > 1024:
                            continue
                        assert lib.ssd_attention_plan(hd, nq, nkv, seqs, rows, positions, 256, plan) == 0
                        wq, wk, chunks = plan
                        assert chunks > 0 and chunks % wk == 0 and (hd, wq, wk) in ((64, 4, 2), (64, 2, 4), (64, 4, 4), (128, 4, 2))
                        forms.add((hd, wq, wk))
    assert len(forms) == 4
    assert lib.ssd_attention_plan(32, 2, 1, 1, 1, 0, 256, plan) == -1 and lib.ssd_attention_plan(64, 3, 2, 1, 1, 0, 256, plan) == -1


def _fits(lib, running, stream, wgs, cus=256):
    return lib.ssd_resident_fits((C.c_int * (2 * len(running) or 1))(*[v for x in running for v in x]), len(running), stream, wgs, cus)


@pytest.mark.parametrize("a,b,fits", [
    (216, 37, 1), (218, 32, 1), (128, 128, 1), (13, 100, 1),                               # 27 + 5, 28 + 4, 16 + 16, 2 + 13 of an XCD's 32 units
    (218, 37, 0), (218, 38, 0), (222, 34, 0), (228, 28, 0), (204, 52, 0),                  # at most 256 together, but 33 on some XCD
    (218, 33, 0), (129, 128, 0), (256, 1, 0)])
def test_launches_run_side_by_side_where_every_xcds_share_fits(lib, a, b, fits):
    assert _fits(lib, [(0, a)], 1, b) == _fits(lib, [(0, b)], 1, a) == fits
    assert _fits(lib, [(0, a)], 0, b) == 1                   # (a stream's launches are ordered among themselves)


def test_a_stream_counts_with_its_largest_launch(lib):
    assert _fits(lib, [], 0, 256) == 1
    assert _fits(lib, [(0, 100), (0, 218), (0, 13)], 1, 32) == 1 and _fits(lib, [(0, 13), (0, 218)], 1, 33) == 0
    assert _fits(lib, [(0, 100), (2, 100), (0, 90), (1, 256)], 1, 48) == 1 and _fits(lib, [(0, 100), (2, 100), (0, 90)], 1, 49) == 0
    assert _fits(lib, [(s, 1) for s in range(31)], 31, 8) == 1 and _fits(lib, [(s, 1) for s in range(32)], 32, 1) == 0
    assert _fits(lib, [(0, 32)], 1, 32, 64) == 1 and _fits(lib, [(0, 33)], 1, 32, 64) == 0
    assert _fits(lib, [], 0, 257) == -1 and _fits(lib, [(0, 0)], 1, 1) == -1 and lib.ssd_resident_fits(None, 1, 0, 1, 256) == -1
