"""Every tile of the wide projection kernel against the any-M path, which shares no matrix code with it: one layer, row
counts and widths at which the launcher takes each of them with either activation format, whole and in runs (test_projection_plan.py
asks the launcher's planner whether these lists still do), with ragged last tiles on both sides."""
import math
from types import SimpleNamespace

import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

VOCAB, BINS = 2048, 256
GENERIC, BATCH = 1, 4

# (batch, K) per width: split activations, single-bf16 activations
_ALL = ((2, 5), (3, 7), (4, 7), (7, 5), (7, 7), (8, 8), (11, 7), (37, 3), (23, 7), (32, 7), (32, 8), (12, 23), (48, 7), (63, 7), (75, 7))
SPLIT_CALLS = {(4096, 11008): _ALL + ((21, 4), (33, 4), (37, 4)), (2048, 5632): _ALL + ((169, 4),), (1024, 2736): _ALL, (512, 1376): ((113, 4),)}
SINGLE_CALLS = {(4096, 11008): ((7, 7), (11, 7), (32, 7), (12, 23), (64, 7), (64, 8), (33, 4)), (2048, 5632): ((33, 4), (41, 4), (225, 4)),
                (512, 1376): ((161, 4), (225, 4)), (5120, 13760): ((81, 4), (129, 4), (145, 4))}


def _model(d, f, seed):
    g = torch.Generator(device="cuda:0").manual_seed(seed)
    rnd = lambda *s: torch.randn(s, generator=g, device="cuda:0").mul_(0.02).to(torch.bfloat16)
    w = {"tok_emb": rnd(VOCAB, d), "lm_head": rnd(VOCAB, d), "final_norm": 1 + 5 * rnd(d).float(),
         "attn_norm": [1 + 5 * rnd(d).float()], "ffn_norm": [1 + 5 * rnd(d).float()]}
    for n, o, i in (("wq", d, d), ("wk", d, d), ("wv", d, d), ("wo", d, d), ("w_gate", f, d), ("w_up", f, d), ("w_down", d, f)):
        w[n] = [rnd(o, i)]
    shape = SimpleNamespace(n_layers=1, d_model=d, n_heads=d // 128, head_dim=128, d_ffn=f, vocab=VOCAB, n_bins=BINS, rms_eps=1e-6,
                            rope_base=10000.0)
    return shape, w


def _run(P, ver, path, batch, K, prefix, seed):
    g = torch.Generator(device="cuda:0").manual_seed(seed)
    s = ver.model.shape
    k, v = (torch.randn((1, batch, s["n_heads"], ver.kv_capacity, 128), generator=g, device="cuda:0").to(torch.bfloat16) for _ in range(2))
    tok = torch.randint(0, VOCAB, (batch, K), generator=g, device="cuda:0", dtype=torch.int32)
    i32 = dict(device="cuda:0", dtype=torch.int32)
    assert P.heisd_verify_set_path(ver.ctx, path) == 0
    out = ver.step(k, v, torch.full((batch,), prefix, **i32), torch.zeros(batch, **i32), tok, P.make_accept_desc(15, 30, (3, 3, 1), 4))
    torch.cuda.synchronize()
    assert P.heisd_verify_check(ver.ctx) == 0
    return out["bin_logits"].double(), k.float(), v.float()


@pytest.mark.parametrize("d,f", list(SPLIT_CALLS))
def test_tiles_against_the_any_m_path(d, f):
    """10 to 676 rows.  Both paths hold activations as a bf16 head and tail (2^-17 of the value) and add in fp32: two orders of
    summation of one layer and the head differ by 1.5e-5, asserted to 6e-5.  A cached value next to a rounding boundary may fall either way:
    one bf16 unit, in few elements; one that nearly cancels is off by what its sum is off by, 1.5e-5 of a value's usual size (20 times that asserted).  d_ffn = 2736 ends in half a k-step; 525 and 676 rows need more row blocks than the others."""
    import paper_2603_17573_amd as P
    shape, w = _model(d, f, d)
    model = P.DeviceModel(shape, w)
    for batch, K in SPLIT_CALLS[d, f]:
        ver = P.Verifier(model, batch, K, 19 + K)
        a, b = (_run(P, ver, p, batch, K, 19, batch) for p in (GENERIC, BATCH))
        rel = ((a[0] - b[0]).norm() / a[0].norm()).item()
        print(d, batch * K, "%.2e" % rel, flush=True)
        assert math.isfinite(rel) and rel < 6e-5, (d, batch, K, rel)
        for x, y in zip(a[1:], b[1:]):
            off = x != y
            assert off.float().mean().item() < 0.01, (d, batch, K)
            assert bool(((x - y).abs() <= x.abs() * 2.0 ** -7 + 3e-4 * x.square().mean().sqrt()).all()), (d, batch, K)


def test_row_scales_of_a_call_of_many_rows():
    """12288 rows: several times as many workgroups as there are compute units, every one of them waiting for its rows' scales; the words come
    from the first workgroups (tolerance as above)."""
    import paper_2603_17573_amd as P
    shape, w = _model(256, 688, 17)
    ver = P.Verifier(P.DeviceModel(shape, w), 512, 24, 40)
    a, b = (_run(P, ver, p, 512, 24, 16, 3) for p in (GENERIC, BATCH))
    rel = ((a[0] - b[0]).norm() / a[0].norm()).item()
    print("%.2e" % rel, flush=True)
    assert math.isfinite(rel) and rel < 6e-5, rel


@pytest.mark.parametrize("d,f,batch,K", [w + c for w, calls in SINGLE_CALLS.items() for c in calls])
def test_tiles_with_single_bf16_activations(d, f, batch, K):
    """One bf16 per activation: every GEMM input is rounded to 2^-9 of its value, so sums of thousands of such terms are off by about
    that over one layer's four projections and the head (measured 4e-3 against split activations); 2e-2 asserted."""
    import paper_2603_17573_amd as P
    shape, w = _model(d, f, 5)
    ver = P.Verifier(P.DeviceModel(shape, w), batch, K, 19 + K)
    a = _run(P, ver, GENERIC, batch, K, 19, batch)
    assert P.heisd_verify_set_activations(ver.ctx, P.binding.HEISD_ACT_BF16) == 0
    b = _run(P, ver, BATCH, batch, K, 19, batch)
    rel = ((a[0] - b[0]).norm() / a[0].norm()).item()
    print(d, batch * K, "%.2e" % rel, flush=True)
    assert math.isfinite(rel) and 1e-4 < rel < 2e-2, rel


@pytest.mark.parametrize("act", ["split", "bf16"])
def test_prefill_of_one_episode_multiplies_the_last_column_tile(act):
    """The LM head of a chunk of one episode runs on the column tile that holds the last row: chunks that end on either side of a
    tile, in a context sized for more rows, against the any-M path's head over all rows (tolerances as above)."""
    import paper_2603_17573_amd as P
    shape, w = _model(512, 1376, 11)
    model = P.DeviceModel(shape, w)
    i32 = dict(device="cuda:0", dtype=torch.int32)
    for n, max_k in ((9, 9), (16, 40), (17, 64), (33, 33), (48, 64), (63, 64), (64, 64), (65, 65), (128, 128), (131, 140)):
        ver = P.Verifier(model, 1, max_k, max_k)
        g = torch.Generator(device="cuda:0").manual_seed(n)
        ids = torch.randint(0, VOCAB, (1, n), generator=g, **i32)
        got = []
        for path in (GENERIC, BATCH):
            assert P.heisd_verify_set_path(ver.ctx, path) == 0
            assert P.heisd_verify_set_activations(ver.ctx, P.binding.HEISD_ACT_BF16 if act == "bf16" and path == BATCH
                                                  else P.binding.HEISD_ACT_SPLIT) == 0
            out = ver.prefill_chunk(*ver.new_cache(1), torch.zeros(1, **i32), token_ids=ids, want_logits=True)
            torch.cuda.synchronize()
            assert P.heisd_verify_check(ver.ctx) == 0
            assert int(out["next_bin"][0]) == int(out["last_logits"][0].argmax())
            got.append(out["last_logits"].double())
        rel = ((got[0] - got[1]).norm() / got[0].norm()).item()
        print(n, act, "%.2e" % rel, flush=True)
        assert math.isfinite(rel) and rel < (2e-2 if act == "bf16" else 6e-5), (n, rel)


@pytest.mark.parametrize("batch,n,bins,act", [(12, 1, 256, "split"), (5, 7, 528, "split"), (3, 40, 48, "split"), (40, 1, 256, "bf16"),
                                              (9, 5, 528, "bf16")])
def test_last_rows_out_of_the_heads_runs(batch, n, bins, act):
    """Decode steps and prefill chunks of several episodes: the last rows' logits are added up from the runs of the LM head (d_model 4096:
    cut), with fewer bins than threads and more, and one episode whose rows do not fit its cache; against the any-M path (tolerances as above)."""
    import paper_2603_17573_amd as P
    shape, w = _model(4096, 1376, 13)
    shape.n_bins = bins
    model = P.DeviceModel(shape, w)
    ver = P.Verifier(model, batch, n, 16 + n)
    i32 = dict(device="cuda:0", dtype=torch.int32)
    g = torch.Generator(device="cuda:0").manual_seed(n)
    ids = torch.randint(0, VOCAB, (batch, n), generator=g, **i32)
    prefix = torch.arange(batch, **i32) % 16
    prefix[batch // 2] = 17
    got = []
    for path in (GENERIC, BATCH):
        assert P.heisd_verify_set_path(ver.ctx, path) == 0
        assert P.heisd_verify_set_activations(ver.ctx, P.binding.HEISD_ACT_BF16 if act == "bf16" and path == BATCH
                                              else P.binding.HEISD_ACT_SPLIT) == 0
        k, v = ver.new_cache(batch)
        out = ver.prefill_chunk(k.fill_(0.5), v.fill_(-0.25), prefix, token_ids=ids, want_logits=True)
        torch.cuda.synchronize()
        assert P.heisd_verify_check(ver.ctx) != 0                    # the episode without room
        fits = torch.arange(batch, device="cuda:0") != batch // 2
        assert int(out["next_bin"][batch // 2]) == -1 and bool(out["last_logits"][batch // 2].isnan().all())
        assert torch.equal(out["next_bin"][fits].long(), out["last_logits"][fits].argmax(1))
        got.append(out["last_logits"][fits].double())
    rel = ((got[0] - got[1]).norm() / got[0].norm()).item()
    print(batch, n, bins, act, "%.2e" % rel, flush=True)
    assert math.isfinite(rel) and rel < (2e-2 if act == "bf16" else 6e-5), rel
