"""How the path for more than 8 rows runs its projections, asked of the library's own planner (no GPU): properties of every launch over
the model widths and row counts it serves."""
import heapq

import pytest

QKV, O, GATEUP, DOWN, HEAD, HEAD_LAST = range(6)
GEMM, NS, TILE = range(3)
CUS = 256


@pytest.fixture(scope="module")
def P():
    import os
    from paper_2603_17573_amd import binding, build
    if not os.path.exists(binding.LIB_PATH):
        build.build(force=False)
    return binding


def desc(P, d, f, max_rows, bins=256):
    """Description of a context of one layer for calls of up to max_rows rows (max_k is 1024 at most)."""
    k = max(i for i in range(1, 1025) if max_rows % i == 0)
    shape = dict(n_layers=1, d_model=d, n_heads=d // 128, head_dim=128, d_ffn=f, vocab=32000, n_bins=bins, bin_token_base=32000 - bins,
                 rms_eps=1e-6, rope_base=1e4)
    ptrs = {n: [4096] for n in ("wq", "wk", "wv", "wo", "w_gate", "w_up", "w_down", "attn_norm", "ffn_norm")}
    ptrs.update(tok_emb=4096, lm_head=4096, final_norm=4096)                 # never dereferenced
    return P.make_model_desc(shape, ptrs, max_rows // k, k, 4096)


def plan(P, de, rows, projection, act=False, cus=CUS):
    rc, p = P.heisd_debug_projection_plan(de[0], cus, rows, act, projection)
    assert rc == 0
    return p


def ffn(d):
    return d * 43 // 16 // 16 * 16


def stuck_at(p, weight_tiles, slots):
    """Workgroups of a launch dispatched, in order, to `slots` places: every workgroup first produces its rows' scales and leaves when
    all rows of its block have theirs.  None if all of them leave, else how many were dispatched when nothing moved any more."""
    rows = p["ct"] * (16 if p["single"] else 8)
    block = p["column_tiles"] * (16 if p["single"] else 8)
    n_blk = -(-p["ct"] // p["column_tiles"])
    groups = -(-weight_tiles // p["weight_tiles"])
    makers = p["scale_workgroups"]

    def needs(wg):                           # the last workgroup this one waits for
        in_xcd = wg >> 3
        if in_xcd // n_blk * 8 + (wg & 7) >= groups:
            return -1
        lo = in_xcd % n_blk * block
        return max(m // p["waves"] % makers for m in range(lo, min(rows, lo + block)))

    there = [needs(wg) for wg in range(min(slots, p["workgroups"]))]
    heapq.heapify(there)
    for wg in range(len(there), p["workgroups"]):
        if there[0] >= wg:
            return wg
        heapq.heapreplace(there, needs(wg))
    return None


@pytest.mark.parametrize("d", [256, 512, 1024, 4096])
def test_nobody_waits_for_a_workgroup_that_is_not_dispatched(P, d):
    """The projections of a normalised input wait inside their launch for words that its first workgroups write.  However many rows
    there are, these are dispatched before anybody waits for ever: on the whole chip, and where launches of
    other streams leave half of it; a quarter is enough for 448 rows on tiles of four and more waves."""
    f = ffn(d)
    for rows in (448, 525, 1200, 2640, 4096, 6001, 11776, 16060, 22042, 40000, 70000):
        de = desc(P, d, f, rows)
        for act in (False, True):
            for projection, tiles in ((QKV, 3 * d // 16), (GATEUP, 2 * f // 16), (HEAD, 16)):
                p = plan(P, de, rows, projection, act)
                if p["kernel"] == TILE and p["runs"] == 1:
                    for slots in (CUS * p["per_unit"], CUS // 2) + ((CUS // 4,) if rows == 448 and p["waves"] > 3 else ()):
                        assert 1 <= p["scale_workgroups"] <= min(slots, p["workgroups"])
                        assert stuck_at(p, tiles, slots) is None, (d, rows, act, projection, slots, p)


def test_the_simulation_sees_a_launch_that_cannot_end(P):
    """Gate/up of 16060 rows with d_model 256 when every workgroup made some rows' words: 64 rows of words for every 112 waited for."""
    p = dict(single=0, ct=2008, weight_tiles=12, column_tiles=14, waves=4, workgroups=1152, scale_workgroups=1152)
    assert stuck_at(p, 2 * 688 // 16, CUS) is not None
    assert stuck_at(dict(p, scale_workgroups=CUS // 4), 2 * 688 // 16, CUS) is None


@pytest.mark.parametrize("d", [256, 1024, 2048])
def test_column_tiles_read_are_inside_the_records(P, d):
    """bat_gemm reads the column tiles of its call at every k-step, the zero k-step behind the last among them: none may lie beyond the
    allocated ones.  The head of a one-episode prefill chunk starts at the last tile in use, which may be the last allocated.  (bat_gemm_wide reads at most
    as many tiles as are allocated, and not at the zero k-step, whose two k-tiles lie behind it.)"""
    for max_rows in (9, 40, 64, 72, 276, 520):
        de = desc(P, d, ffn(d), max_rows)
        for rows in range(1, max_rows + 1):
            for projection in range(6):
                p = plan(P, de, rows, projection)
                if p["kernel"] == GEMM:
                    assert p["column_tiles"] == p["ct"] and p["first_ct"] + p["column_tiles"] <= p["cts"], (rows, max_rows, projection, p)


def test_few_rows_of_a_long_reduction_fill_the_units(P):
    """Down projection of 41 to 64 rows, d_ffn 11008.  With two workgroups per compute unit both of a weight group's row blocks fetch its weights from
    memory; 8 x 4 tiles in seven runs, which leave one place in eight empty, took 36 us with the finishing launch, whole rounds 34."""
    de = desc(P, 4096, 11008, 64)
    for rows in range(41, 65):
        p = plan(P, de, rows, DOWN)
        assert p["kernel"] == TILE and p["workgroups"] in (CUS, 2 * CUS), (rows, p)


def test_a_projection_of_many_weight_tiles_and_a_short_reduction_is_not_cut(P):
    """QKV of 17 to 40 rows, d_model 2048: in runs on tiles, with a launch that adds them, steps of 25 to 32 rows were 1 % slower than before there
    were tiles; whole on bat_gemm 3 % faster."""
    de = desc(P, 2048, 5504, 40)
    for rows in range(9, 41):
        assert plan(P, de, rows, QKV)["kernel"] == GEMM, rows
    assert plan(P, de, 32, O)["kernel"] == plan(P, de, 32, DOWN)["kernel"] == TILE


def test_blocks_of_sixteen_column_tiles(P):
    """512 rows of single-bf16 activations (32 column tiles) and 600 rows at d_model 3072 are whole blocks of 16 or nearly: on blocks of 14 and 9
    steps of two layers were 3 % slower than before there were tiles."""
    for d, f, rows, projection, act in ((4096, 11008, 512, GATEUP, True), (4096, 11008, 512, DOWN, True), (3072, 8192, 600, GATEUP, False),
                                        (4096, 11008, 256, GATEUP, False)):
        p = plan(P, desc(P, d, f, 1024), rows, projection, act)
        assert (p["weight_tiles"], p["column_tiles"]) == (12, 16), (d, rows, p)


def kernels(P, d, f, rows, act):
    """What the projections of a call run on: the tile and whether its reduction is cut, or the kernel of few rows and its size."""
    de, out = desc(P, d, f, rows), set()
    for projection in range(HEAD + 1):
        p = plan(P, de, rows, projection, act)
        if p["kernel"] == TILE:
            out.add(("tile", p["weight_tiles"], p["column_tiles"], p["waves"], p["single"], p["runs"] > 1))
        else:
            out.add((p["kernel"], p["single"], p["ct"] if p["kernel"] == GEMM else p["weight_tiles"]))
    return out


def test_the_gpu_tests_run_every_kernel_there_is(P):
    """Whatever tile the planner takes for some call of 9 to 1028 rows at the usual widths, with either activation format, whole or in runs: one
    of the calls that the GPU tests compare with the any-M path takes it too."""
    import test_gpu_tiles as G
    run, there = set(), set()
    for act, calls in ((False, G.SPLIT_CALLS), (True, G.SINGLE_CALLS)):
        for (d, f), rows in calls.items():
            for batch, k in rows:
                run |= kernels(P, d, f, batch * k, act)
    for d in (256, 512, 768, 1024, 1536, 2048, 3072, 4096, 5120):
        for rows in list(range(9, 130)) + list(range(132, 1030, 4)):
            there |= kernels(P, d, ffn(d), rows, False) | (kernels(P, d, ffn(d), rows, True) if rows > 32 else set())
    assert len([k for k in there if k[0] == "tile"]) > 60
    assert not there - run, sorted(there - run, key=str)
