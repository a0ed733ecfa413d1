"""The work that users of this library have it do, as measurable cases over its real range.

Every case goes through the public entry points: the verify step (one to 64 episodes, linear drafts and draft
trees), the autoregressive decode step, the chunked prefill, the retrieval search and the offline stage of the
verify-skip decision.  The decoder cases have the width of the 7B backbone (d_model 4096, 32 heads of 128,
d_ffn 11008).  One of them, the single-episode verify step, runs all 32 layers; the others run a slice of four
layers with the LM-head slice and the acceptance behind it (1.6 GB of weights: far more than any cache holds),
so that rounding in one layer does not travel through 32 of them.  Weights, caches and drafts are random and
seeded.

prepare() builds what a user's program holds: the weights in HBM, a context, the episodes' caches and the arrays
of one call.  run() is that call.  exact() is the same forward in 64 bits, in plain torch.
"""
import math
from types import SimpleNamespace

import torch

import paper_2603_17573_amd as P

DEV = "cuda:0"
VOCAB, BINS = 32000, 256
EPS, ROPE_BASE = 1e-6, 10000.0
GROUPS, EXACT_MASK = (3, 3, 1), 0b100            # (X,Y,Z), (rX,rY,rZ), gripper


def _decoder(name, kind, batch, k, prefix, **more):
    c = dict(name=name, kind=kind, layers=4, heads=32, head_dim=128, d_ffn=11008, batch=batch, k=k, prefix=prefix,
             ragged=False, skip=0.0, act="split")
    c.update(more)
    return c


def listed():
    return [
        # A two-layer toy policy, one episode: the step is a dozen launches of almost no work (launch latency).
        _decoder("verify_tiny", "verify", 1, 7, 64, layers=2, heads=4, head_dim=64, d_ffn=688),
        # The headline: one robot, one action of seven drafted tokens, the whole 7B model, a 276-row prefix.
        _decoder("verify_1", "verify", 1, 7, 276, layers=32),
        # The fallback of speculative decoding: one token, one episode (every candidate was rejected).
        _decoder("decode_1", "decode", 1, 1, 276),
        # Eight robots (or simulator instances) verified together.
        _decoder("verify_8", "verify", 8, 7, 276),
        # Sixteen episodes, two-action drafts, episodes at different positions, three in ten skip verification.
        _decoder("verify_16_ragged", "verify", 16, 14, 532, ragged=True, skip=0.3),
        # A full simulator batch: 64 episodes, 448 rows.
        _decoder("verify_64", "verify", 64, 7, 276),
        # The same with one bf16 per activation, the precision the paper runs its models in.
        _decoder("verify_64_bf16", "verify", 64, 7, 276, act="bf16"),
        # A draft tree of four retrieved candidates (4 x 3 + 16 x 3 + 16 tokens), one episode.
        _decoder("tree_4", "tree", 1, 76, 276),
        # A new observation: 256 visual rows and 20 prompt tokens into an empty cache, one chunk.
        _decoder("prefill_276", "prefill", 1, 276, 0),
        # One query against the paper-sized database (273465 embeddings of 4352), four candidates.
        dict(name="retrieve_1", kind="retrieve", n=273465, d=4352, batch=1, k=4),
        # The same for the 64 episodes of a full simulator batch.
        dict(name="retrieve_64", kind="retrieve", n=273465, d=4352, batch=64, k=4),
        # The offline stage of the skip decision: similarities of all pairs of 300 trajectory points.
        dict(name="skip_offline", kind="skip", n=300, d=4096, threshold=0.8),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["verify", "verify", "verify", "verify", "decode", "tree", "prefill", "prefill", "retrieve", "retrieve",
                       "skip"])
    if kind == "retrieve":
        return dict(kind=kind, n=_log(rng, 1000, 273465), d=4 * _log(rng, 128, 1088), batch=_log(rng, 1, 64), k=_log(rng, 1, 32))
    if kind == "skip":
        return dict(kind=kind, n=_log(rng, 16, 400), d=4 * _log(rng, 64, 1024), threshold=round(rng.uniform(0.5, 0.95), 3))
    head_dim = rng.choice([64, 128, 128, 128])
    heads = rng.choice([4, 8, 12, 16, 24, 32]) if head_dim == 128 else rng.choice([4, 8, 16, 32])
    d = heads * head_dim
    c = _decoder("", kind, 1, 1, _log(rng, 16, 1000), layers=rng.choice([1, 2, 3]), heads=heads, head_dim=head_dim,
                 d_ffn=16 * int(round(d * rng.uniform(2.5, 3.0) / 16)), ragged=rng.random() < 0.5,
                 act=rng.choice(["split", "split", "bf16"]))
    del c["name"]
    if kind == "verify":
        c["k"] = rng.choice([3, 6, 7, 7, 7, 14, 21])
        c["batch"] = max(1, min(_log(rng, 1, 64), 448 // c["k"]))
        c["skip"] = rng.choice([0.0, 0.0, 0.3])
    elif kind == "decode":
        c["batch"] = _log(rng, 1, 64)
    elif kind == "tree":
        r = rng.choice([2, 3, 4, 5])
        c["k"] = 3 * r + 3 * r * r + r * r                        # candidates that share nothing
        c["batch"] = rng.choice([1, 1, 2, 3, 4]) if r > 2 else rng.choice([1, 2, 4, 8])
    else:
        c["k"], c["prefix"] = _log(rng, 16, 400), rng.choice([0, 0, _log(rng, 16, 500)])
    return c


# ---- inputs ---------------------------------------------------------------------------------------------------

def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(seed)


def _normal(g, shape, std, dtype=torch.bfloat16):
    return torch.randn(shape, generator=g, device=DEV, dtype=dtype).mul_(std)


def _shape(c):
    return SimpleNamespace(n_layers=c["layers"], d_model=c["heads"] * c["head_dim"], n_heads=c["heads"], head_dim=c["head_dim"],
                           d_ffn=c["d_ffn"], vocab=VOCAB, n_bins=BINS, rms_eps=EPS, rope_base=ROPE_BASE)


def _weights(c, seed):
    sh, g = _shape(c), _gen(seed * 8 + 1)
    d, f, n = sh.d_model, sh.d_ffn, sh.n_layers
    w = {"tok_emb": _normal(g, (VOCAB, d), 0.02), "lm_head": _normal(g, (VOCAB, d), 0.02)}
    for name, o, i in (("wq", d, d), ("wk", d, d), ("wv", d, d), ("wo", d, d), ("w_gate", f, d), ("w_up", f, d), ("w_down", d, f)):
        w[name] = [_normal(g, (o, i), 0.02) for _ in range(n)]
    for name in ("attn_norm", "ffn_norm"):
        w[name] = [1 + _normal(g, (d,), 0.1, torch.float32) for _ in range(n)]
    w["final_norm"] = 1 + _normal(g, (d,), 0.1, torch.float32)
    return w


def _tree_parents(k):
    """Parents of the draft tree of r candidates that share nothing (k = 3r + 3r^2 + r^2 tokens), depth first."""
    r = next(r for r in range(1, 16) if 4 * r * r + 3 * r == k)
    parent = []

    def chain(n, prev):
        for _ in range(n):
            parent.append(prev)
            prev = len(parent) - 1
        return prev

    for _ in range(r):
        a = chain(3, -1)
        for _ in range(r):
            chain(1, chain(3, a))
    return parent


def _calls(c, seed):
    """The arrays of one call (caches, positions, tokens), from the seed alone."""
    g, b, k, d = _gen(seed * 8 + 2), c["batch"], c["k"], c["heads"] * c["head_dim"]
    cap = c["prefix"] + k
    s = SimpleNamespace()
    std = 0.02 * math.sqrt(d)                                     # the scale a random model gives its keys and values
    s.k_cache = _normal(g, (c["layers"], b, c["heads"], cap, c["head_dim"]), std)
    s.v_cache = _normal(g, (c["layers"], b, c["heads"], cap, c["head_dim"]), std)
    plen = torch.full((b,), c["prefix"], device=DEV, dtype=torch.int32)
    if c["ragged"] and c["prefix"]:
        plen -= torch.randint(0, c["prefix"] // 2 + 1, (b,), generator=g, device=DEV, dtype=torch.int32)
    s.prefix_len = plen
    s.first_pred = torch.randint(0, BINS, (b,), generator=g, device=DEV, dtype=torch.int32)
    s.tokens = VOCAB - BINS + torch.randint(0, BINS, (b, k), generator=g, device=DEV, dtype=torch.int32)
    # a retrieved draft begins close to what the target wants: the first token two bins from its prediction
    s.tokens[:, 0] = VOCAB - BINS + (s.first_pred + 2).clamp(max=BINS - 1)
    s.skip = (torch.rand((b,), generator=g, device=DEV) < c["skip"]).to(torch.uint8) if c["skip"] else None
    s.rows, s.parent = None, None
    if c["kind"] == "prefill":                                    # visual rows as embeddings, then prompt ids
        visual = max(1, k * 12 // 13)
        s.tokens = torch.randint(0, VOCAB - BINS, (b, k), generator=g, device=DEV, dtype=torch.int32)
        s.tokens[:, :visual] = -1
        s.rows = torch.randn((b, k, d), generator=g, device=DEV)
    if c["kind"] == "tree":
        s.parent = torch.tensor(_tree_parents(k), device=DEV, dtype=torch.int32).repeat(b, 1)
    return s


def _vectors(c, seed):
    """A database of L2-normalised embeddings with payload, and queries close to stored entries."""
    g, n, d, b = _gen(seed * 8 + 3), c["n"], c["d"], c["batch"]
    s = SimpleNamespace()
    s.db = torch.empty((n, d), device=DEV, dtype=torch.bfloat16)
    for i in range(0, n, 32768):
        x = torch.randn((min(32768, n - i), d), generator=g, device=DEV)
        s.db[i:i + 32768] = x / x.norm(dim=1, keepdim=True)
    near = torch.randint(0, n, (b,), generator=g, device=DEV)
    q = s.db[near].float() + torch.randn((b, d), generator=g, device=DEV) * (0.5 / math.sqrt(d))
    s.queries = q / q.norm(dim=1, keepdim=True)
    s.payload = torch.randint(0, BINS, (n, 7), generator=g, device=DEV, dtype=torch.int32)
    return s


def _trajectory(c, seed):
    """Features of trajectory points that drift: nearby points are similar."""
    g = _gen(seed * 8 + 4)
    f = torch.randn((c["n"], c["d"]), generator=g, device=DEV)
    f[1:] *= 0.1
    return torch.cumsum(f.double(), 0).float()


def prepare(case, seed):
    c = case
    if c["kind"] == "retrieve":
        s = _vectors(c, seed)
        s.out = {"index": torch.empty((c["batch"], c["k"]), device=DEV, dtype=torch.int32),
                 "score": torch.empty((c["batch"], c["k"]), device=DEV),
                 "payload": torch.empty((c["batch"], c["k"], 7), device=DEV, dtype=torch.int32)}
        s.workspace = torch.empty(P.heisd_retrieve_workspace_bytes(c["n"], c["batch"], c["k"]), device=DEV, dtype=torch.uint8)
        s.case = c
        return s
    if c["kind"] == "skip":
        s = SimpleNamespace(case=c, feat=_trajectory(c, seed), work=torch.empty(1, device=DEV, dtype=torch.int64))
        s.out = {"similarity": torch.empty((c["n"], c["n"]), device=DEV), "min_s": torch.empty(1, device=DEV),
                 "o_dist": torch.empty(1, device=DEV, dtype=torch.int32)}
        return s
    s = _calls(c, seed)
    s.case = c
    s.verifier = P.Verifier(P.DeviceModel(_shape(c), _weights(c, seed), DEV), c["batch"], c["k"], c["prefix"] + c["k"])
    if c["act"] == "bf16" and P.heisd_verify_set_activations(s.verifier.ctx, P.binding.HEISD_ACT_BF16) != 0:
        raise RuntimeError("activation format refused")
    s.accept = P.make_accept_desc(15, 30, GROUPS, EXACT_MASK)
    b, k = c["batch"], c["k"]
    i32 = dict(device=DEV, dtype=torch.int32)
    if c["kind"] in ("verify", "tree"):
        s.out = {"accepted_len": torch.empty(b, **i32), "next_token": torch.empty(b, **i32),
                 "target_bins": torch.empty((b, k + 1), **i32), "bin_logits": torch.empty((b, k, BINS), device=DEV)}
        if c["kind"] == "tree":
            s.out["accepted_path"] = torch.empty((b, k), **i32)
    else:
        s.out = {"next_bin": torch.empty(b, **i32), "last_logits": torch.empty((b, BINS), device=DEV)}
    return s


def run(state):
    s, c = state, state.case
    if c["kind"] == "retrieve":
        o, st = s.out, torch.cuda.current_stream().cuda_stream
        rc = P.heisd_retrieve_topk(s.db.data_ptr(), c["n"], c["d"], s.queries.data_ptr(), c["batch"], c["k"], s.payload.data_ptr(), 7,
                                   o["index"].data_ptr(), o["score"].data_ptr(), o["payload"].data_ptr(), s.workspace.data_ptr(),
                                   s.workspace.numel(), st)
        if rc != 0:
            raise RuntimeError("heisd_retrieve_topk: %d" % rc)
        return o
    if c["kind"] == "skip":
        o, st = s.out, torch.cuda.current_stream().cuda_stream
        rc = P.heisd_skip_offline(s.feat.data_ptr(), c["n"], c["d"], c["threshold"], o["similarity"].data_ptr(), s.work.data_ptr(),
                                  o["min_s"].data_ptr(), o["o_dist"].data_ptr(), st)
        if rc != 0:
            raise RuntimeError("heisd_skip_offline: %d" % rc)
        return o
    v = s.verifier
    if c["kind"] == "verify":
        out = v.step(s.k_cache, s.v_cache, s.prefix_len, s.first_pred, s.tokens, s.accept, s.skip, out=s.out)
    elif c["kind"] == "tree":
        out = v.tree_step(s.k_cache, s.v_cache, s.prefix_len, s.first_pred, s.tokens, s.parent, s.accept, out=s.out)
    else:
        out = v.prefill_chunk(s.k_cache, s.v_cache, s.prefix_len, token_ids=s.tokens, x_rows=s.rows, want_logits=True, out=s.out)
    return dict(out, k_cache=s.k_cache, v_cache=s.v_cache)


def work(case):
    """What one pass cannot do without: every weight, cached row and input once, every output once."""
    c = case
    if c["kind"] == "retrieve":
        n, d, b, k = c["n"], c["d"], c["batch"], c["k"]
        return {"bytes": 2 * n * d + 4 * b * d + b * k * (8 + 2 * 4 * 7), "flops": 2 * n * d * b}
    if c["kind"] == "skip":
        n, d = c["n"], c["d"]
        return {"bytes": 4 * n * d + 4 * n * n + 8, "flops": n * (n + 1) * d}
    d, f, layers = c["heads"] * c["head_dim"], c["d_ffn"], c["layers"]
    active = c["batch"] * (1 - c["skip"])
    prefix = c["prefix"] - (c["prefix"] // 4 if c["ragged"] else 0)          # the mean
    rows = active * c["k"]
    per_layer = 4 * d * d + 3 * d * f
    heads = rows if c["kind"] in ("verify", "tree") else active              # rows whose logits are wanted
    nbytes = layers * (2 * per_layer + 8 * d + 4 * d * (active * prefix + rows)) + 2 * BINS * d \
        + rows * d * (4 if c["kind"] == "prefill" else 2) + heads * BINS * 4
    flops = layers * (2 * per_layer * rows + 4 * d * rows * (prefix + c["k"] / 2)) + 2 * BINS * d * heads
    return {"bytes": int(nbytes), "flops": int(flops)}


def tolerance(case):
    c = case
    if c["kind"] in ("retrieve", "skip"):
        return {"rel": 1e-5, "max": 1e-4, "differ": 0.01}
    if c["act"] == "bf16" and c["batch"] * c["k"] > 32:
        return {"rel": 1.5e-2, "max": 2e-1, "differ": 0.01}
    # logits differ by 1.5e-5 between two orders of summation; the cache is bf16, where a value next to a rounding
    # boundary may fall either way (one unit is up to 2^-7 of it; 1.4e-4 in all in a prefill, whose cache is all new)
    return {"rel": 6e-4, "max": 1.6e-2, "differ": 0.01}


# ---- the same in 64 bits --------------------------------------------------------------------------------------

def _rms64(x, gain):
    return x * torch.rsqrt(x.square().mean(-1, keepdim=True) + EPS) * gain.double()


def _rope64(x, pos, head_dim):
    """x [B, H, T, head_dim], pos [B, T]; rotate-half pairing."""
    half = head_dim // 2
    theta = ROPE_BASE ** (-2.0 * torch.arange(half, device=DEV, dtype=torch.float64) / head_dim)
    ang = pos.double()[:, None, :, None] * theta
    a, b = x[..., :half], x[..., half:]
    return torch.cat([a * ang.cos() - b * ang.sin(), b * ang.cos() + a * ang.sin()], -1)


def _forward64(c, w, s):
    """Final hidden states [B, T, d] and the caches with the new rows in place, in 64 bits."""
    b, t, heads, hd = c["batch"], c["k"], c["heads"], c["head_dim"]
    d = heads * hd
    live = s.skip.eq(0) if s.skip is not None else torch.ones(b, dtype=torch.bool, device=DEV)
    x = w["tok_emb"][s.tokens.long().clamp(min=0)].double()
    if s.rows is not None:
        x = torch.where((s.tokens < 0)[..., None], s.rows.double(), x)
    plen = s.prefix_len.long()
    if s.parent is None:
        depth = torch.arange(t, device=DEV)
        sees = depth[None, :] <= depth[:, None]                              # causal inside the block
    else:
        sees = torch.eye(t, dtype=torch.bool, device=DEV)
        depth = torch.zeros(t, dtype=torch.long, device=DEV)
        for i, p in enumerate(s.parent[0].tolist()):
            if p >= 0:
                sees[i] |= sees[p]
                depth[i] = depth[p] + 1
    pos = plen[:, None] + depth[None, :]
    old = torch.arange(c["prefix"], device=DEV)[None, :] < plen[:, None]     # [B, prefix]
    mask = torch.cat([old[:, None, :].expand(b, t, -1), sees[None].expand(b, t, t)], -1)
    at = (plen[:, None] + torch.arange(t, device=DEV))[:, None, :, None].expand(b, heads, t, hd)
    caches = [s.k_cache.double(), s.v_cache.double()]
    for l in range(c["layers"]):
        h = _rms64(x, w["attn_norm"][l])
        q, k, v = ((h @ w[n][l].double().T).view(b, t, heads, hd).transpose(1, 2) for n in ("wq", "wk", "wv"))
        q, k = _rope64(q, pos, hd), _rope64(k, pos, hd)
        keys = torch.cat([caches[0][l, :, :, :c["prefix"]], k], 2)
        values = torch.cat([caches[1][l, :, :, :c["prefix"]], v], 2)
        p = torch.matmul(q, keys.transpose(2, 3).contiguous()) / math.sqrt(hd)
        p = torch.softmax(p.masked_fill(~mask[:, None], -math.inf), -1)
        o = torch.matmul(p, values).transpose(1, 2).reshape(b, t, d)
        for cache, new in zip(caches, (k, v)):
            now = cache[l].scatter(2, at, new)
            cache[l] = torch.where(live[:, None, None, None], now, cache[l])
        x = x + o @ w["wo"][l].double().T
        h = _rms64(x, w["ffn_norm"][l])
        a = torch.nn.functional.silu(h @ w["w_gate"][l].double().T) * (h @ w["w_up"][l].double().T)
        x = x + a @ w["w_down"][l].double().T
    logits = _rms64(x, w["final_norm"]) @ w["lm_head"][VOCAB - BINS:].double().T
    logits[~live] = math.nan
    return logits, caches[0], caches[1]


def exact(case, seed):
    c = case
    if c["kind"] == "retrieve":
        s = _vectors(c, seed)
        scores = torch.cat([s.queries.double() @ s.db[i:i + 32768].double().T for i in range(0, c["n"], 32768)], 1)
        return {"index": None, "score": scores.topk(min(c["k"], c["n"]), 1).values, "payload": None}
    if c["kind"] == "skip":
        f = _trajectory(c, seed).double()
        f = f / f.norm(dim=1, keepdim=True)
        sim = f @ f.T
        later = torch.triu(sim, 1)
        above = later[later > c["threshold"]]
        return {"similarity": sim, "min_s": above.min().reshape(1) if above.numel() else torch.full((1,), math.inf, dtype=torch.float64),
                "o_dist": None}
    s = _calls(c, seed)
    logits, k_cache, v_cache = _forward64(c, _weights(c, seed), s)
    if c["kind"] == "verify":
        return {"accepted_len": None, "next_token": None, "target_bins": None, "bin_logits": logits, "k_cache": k_cache,
                "v_cache": v_cache}
    if c["kind"] == "tree":                      # the accepted chain's rows move to the front: where to depends on whole numbers
        return {"accepted_len": None, "next_token": None, "target_bins": None, "bin_logits": logits, "accepted_path": None,
                "k_cache": None, "v_cache": None}
    return {"next_bin": None, "last_logits": logits[:, -1], "k_cache": k_cache, "v_cache": v_cache}
