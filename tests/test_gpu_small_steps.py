"""Steps of at most eight rows at the edges of their kernels: the one-launch-per-phase path (short reductions, one unit per workgroup)
against the persistent kernel, which goes through the same sums on the rings of long reductions, and against the any-M path, which
shares no code with either."""
import math
from types import SimpleNamespace

import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

VOCAB, BINS = 1024, 256
GENERIC, FAST, PERSIST = 1, 2, 3


def _model(P, d, hd, f, layers):
    g = torch.Generator(device="cuda:0").manual_seed(d + f)
    rnd = lambda *s: torch.randn(s, generator=g, device="cuda:0").mul_(0.02).to(torch.bfloat16)
    w = {"tok_emb": rnd(VOCAB, d), "lm_head": rnd(VOCAB, d), "final_norm": 1 + 5 * rnd(d).float()}
    for n in ("attn_norm", "ffn_norm"):
        w[n] = [1 + 5 * rnd(d).float() for _ in range(layers)]
    for n, o, i in (("wq", d, d), ("wk", d, d), ("wv", d, d), ("wo", d, d), ("w_gate", f, d), ("w_up", f, d), ("w_down", d, f)):
        w[n] = [rnd(o, i) for _ in range(layers)]
    shape = SimpleNamespace(n_layers=layers, d_model=d, n_heads=d // hd, head_dim=hd, d_ffn=f, vocab=VOCAB, n_bins=BINS, rms_eps=1e-6,
                            rope_base=10000.0)
    return P.DeviceModel(shape, w)


def _step(P, ver, path, batch, k, prefixes, skip=None):
    s = ver.model.shape
    g = torch.Generator(device="cuda:0").manual_seed(sum(prefixes) + k)
    kc, vc = (torch.randn((s["n_layers"], batch, s["n_heads"], ver.kv_capacity, s["head_dim"]), generator=g, device="cuda:0").to(torch.bfloat16)
              for _ in range(2))
    tok = VOCAB - BINS + torch.randint(0, BINS, (batch, k), generator=g, device="cuda:0", dtype=torch.int32)
    i32 = dict(device="cuda:0", dtype=torch.int32)
    assert P.heisd_verify_set_path(ver.ctx, path) == 0
    out = ver.step(kc, vc, torch.tensor(prefixes, **i32), torch.zeros(batch, **i32), tok, P.make_accept_desc(15, 30, (3, 3, 1), 4), skip)
    torch.cuda.synchronize()
    assert P.heisd_verify_check(ver.ctx) == 0
    return dict({n: t.clone() for n, t in out.items()}, k_cache=kc, v_cache=vc)


def _same_cache(a, c, k, prefixes, skip):
    """Rows that are not the step's are the same bits; an appended element may be rounded the other way (one bf16 unit, up to 2^-7 of it)
    where the two paths' fp32 values, 1e-4 of the row apart at most, lie on two sides of a boundary."""
    for n in ("k_cache", "v_cache"):
        new = torch.zeros(a[n].shape[1:4:2], dtype=torch.bool, device=a[n].device)          # [episode, cache row]
        for e, p in enumerate(prefixes):
            if skip is None or not skip[e]:
                new[e, p:p + k] = True
        x, y = (t[n].double().transpose(2, 3) for t in (a, c))                               # [layer, episode, row, head, channel]
        assert torch.equal(x[:, ~new], y[:, ~new]), n
        x, y = x[:, new], y[:, new]
        off = (x - y).abs() - 2.0 ** -7 * y.abs() - 1e-4 * y.abs().amax((-2, -1), keepdim=True)
        assert off.max().item() <= 0, (n, prefixes, off.max().item())


def _compare(P, ver, batch, k, prefixes, skip=None):
    a, b, c = (_step(P, ver, p, batch, k, prefixes, skip) for p in (FAST, PERSIST, GENERIC))
    for n in a:
        assert torch.equal(a[n].nan_to_num(nan=-7.0), b[n].nan_to_num(nan=-7.0)), (n, batch, k, prefixes)
    _same_cache(a, c, k, prefixes, skip)
    # a greedy bin is the same wherever the best two logits are further apart than the two paths' rows (6e-5 of their norm: below)
    top = c["bin_logits"].double().nan_to_num().topk(2, -1).values
    clear = top[..., 0] - top[..., 1] > 2 * 6e-5 * c["bin_logits"].double().nan_to_num().norm(dim=-1)
    assert torch.equal(a["target_bins"][:, 1:][clear], c["target_bins"][:, 1:][clear]), (batch, k, prefixes)
    x, y = a["bin_logits"].double().nan_to_num(), c["bin_logits"].double().nan_to_num()
    rel = ((x - y).norm() / y.norm()).item()
    print(batch, k, prefixes, "%.2e" % rel, flush=True)
    assert math.isfinite(rel) and rel < 6e-5, (rel, batch, k, prefixes)      # two orders of fp32 sums over bf16 heads and tails: 1.5e-5


@pytest.mark.parametrize("d,hd,f", [(64, 64, 16), (128, 128, 48), (256, 64, 688), (320, 64, 1040), (640, 128, 2064), (1088, 64, 2864),
                                    (1536, 128, 4128), (2048, 128, 5504), (256, 64, 8192), (256, 64, 8208)])
def test_short_reductions(d, hd, f):
    """Reductions of 1 to 172 k-steps (less than one per wave; kernels of one, two, four and eight steps per wave, full and not; d_ffn above 4096
    streams its down projection), more units than compute units, and gate/up of 512 and 513 units: the most that runs one unit per workgroup
    with 256 compute units, and the least that stays on the ring for its units alone."""
    import paper_2603_17573_amd as P
    ver = P.Verifier(_model(P, d, hd, f, 1), 2, 8, 32)
    for batch, k in ((1, 1), (1, 7), (2, 4), (1, 8)):
        _compare(P, ver, batch, k, [21, 13][:batch])


@pytest.mark.parametrize("hd", [64, 128])
def test_prefixes_at_the_edges_of_the_attention_units(hd):
    """Key tiles of 16, the keys requested ahead (384), streams of 32 or 64 value rows and the rows requested ahead (320 or 640); an empty
    prefix; a skipped episode beside a verified one."""
    import paper_2603_17573_amd as P
    ver = P.Verifier(_model(P, 2 * hd, hd, 352, 1), 2, 8, 1411)
    for p in (0, 1, 15, 16, 17, 31, 33, 64, 65, 319, 320, 321, 383, 385, 639, 640, 641, 700, 1300):
        _compare(P, ver, 1, 8 if p % 2 else 7, [p])
    skip = torch.tensor([1, 0], dtype=torch.uint8, device="cuda:0")
    _compare(P, ver, 2, 4, [1403, 321], skip)
    _compare(P, ver, 2, 1, [5, 1000])
