"""Parity of heisd_verify_tree_step (through the C ABI) with the chain-by-chain oracle of
sequence-wise tree verification (paper Sec. 4.2) on the same seeded inputs."""
import numpy as np
import pytest

import oracle
import synth
from helpers import oracle_model, oracle_prefix_cache, teacher_forced_drafts

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

MID = synth.ModelShape(n_layers=3, d_model=512, n_heads=4, head_dim=128, d_ffn=1376, vocab=2048)
SMALL64 = synth.ModelShape(n_layers=2, d_model=256, n_heads=4, head_dim=64, d_ffn=688, vocab=1024)


def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def retrieved_candidates(om, wl, kb, vb, plen, first, R, p_geo):
    """R candidate drafts per episode (stand-ins for Top-K retrieval): the target's own continuation
    (teacher forced) plus seeded geometric offsets per candidate, so that some sequences pass the
    relaxed rule and others do not.  Returns bins i32 [B, R, K]."""
    off = synth.make_candidate_offsets(wl, R, p_geo)
    return np.stack([teacher_forced_drafts(om, wl, kb, vb, plen, first, off[:, r]) for r in range(R)], axis=1)


def padded_trees(P, cands, rule, T=None):
    """Builds every episode's tree with the library's host builder and pads to a common T."""
    from gpu_harness import accept_desc_of
    trees = [P.build_sequence_tree(c, accept_desc_of(rule), 256) for c in cands]
    T = T or max(len(t[0]) for t in trees)
    tokens = np.zeros((len(trees), T), np.int32)
    parent = np.full((len(trees), T), -2, np.int32)
    for b, (tok, par) in enumerate(trees):
        tokens[b, :len(tok)], parent[b, :len(par)] = tok, par
    return tokens, parent


def run_tree_case(wl, R, rule, p_geo=0.5, skip=None, path=0, plen_override=None, extra_rows=0):
    import paper_2603_17573_amd as P
    from gpu_harness import run_gpu_tree_step, compare_tree_with_oracle
    _need_gpu()
    sh = wl.shape
    weights = synth.make_weights(sh, wl.seed)
    om = oracle_model(sh, weights)
    cap0 = wl.prefix_len + wl.K
    kb, vb, plen, first = oracle_prefix_cache(om, wl, cap0)
    if plen_override is not None:
        plen = np.asarray(plen_override, np.int32)
    cands = sh.bin_base + retrieved_candidates(om, wl, kb, vb, plen, first, R, p_geo)
    tokens, parent = padded_trees(P, cands, rule)
    for b in range(wl.batch):                                # the library's builder against the oracle's
        t_ref, p_ref = oracle.build_sequence_tree(cands[b], rule, 256)
        assert tokens[b, :len(t_ref)].tolist() == t_ref.tolist() and parent[b, :len(p_ref)].tolist() == p_ref.tolist()
    T = tokens.shape[1]
    cap = int(max(plen)) + T + 3 + extra_rows
    kb2 = np.zeros(kb.shape[:3] + (cap, kb.shape[4]), np.uint16)
    vb2 = np.zeros_like(kb2)
    kb2[:, :, :, :cap0], vb2[:, :, :, :cap0] = kb, vb
    # rows past the prefix hold a recognisable pattern: the step must not depend on them
    kb2[:, :, :, cap0:], vb2[:, :, :, cap0:] = 0x3F80, 0xBF80
    ref = oracle.verify_tree_step(om, kb2, vb2, plen, first, tokens, parent, rule, skip)
    got = run_gpu_tree_step(sh, weights, kb2, vb2, plen, first, tokens, parent, rule, skip, path=path)
    stats = compare_tree_with_oracle(got, ref, tokens, parent, rule, sh, kb2, vb2, plen, first, skip)
    print(wl.name, "R", R, "T", T, "path", path, stats, "accepted", got["accepted_len"].tolist(),
          ref["accepted_len"].tolist(), flush=True)
    return got, ref, stats, tokens, parent


@pytest.mark.parametrize("path", [0, 1, 4])
def test_c0_shape_top3_tree(path):
    wl = synth.WORKLOADS["C0"]
    got, ref, stats, tokens, parent = run_tree_case(wl, 3, oracle.AcceptRule(wl.tau_tok, wl.tau_seq), path=path)
    assert stats["max_logit_err_over_range"] < 3e-2


def test_mid_shape_batch_with_padding_skip_and_ragged_prefixes():
    wl = synth.Workload("tree_mid", MID, 30, 11, MID.bin_base, batch=3, K=7, draft=("geometric", 0.5), seed=17)
    skip = np.array([0, 1, 0], np.uint8)
    run_tree_case(wl, 3, oracle.AcceptRule(2, 6), p_geo=0.6, skip=skip, plen_override=[41, 17, 33])


def test_two_action_slices_k14_more_than_64_tokens():
    """K = 14 candidates: the tree is capped by the token budget well past one 64-bit mask word."""
    wl = synth.Workload("tree_k14", SMALL64, 0, 20, SMALL64.bin_base, batch=2, K=14, draft=("geometric", 0.5), seed=23)
    got, ref, stats, tokens, parent = run_tree_case(wl, 4, oracle.AcceptRule(2, 6), p_geo=0.7)
    assert tokens.shape[1] > 128


@pytest.mark.parametrize("rule", [oracle.AcceptRule(0, 0), oracle.AcceptRule(15, 30),
                                  oracle.AcceptRule(2, 3, mode=1),
                                  oracle.AcceptRule(1, 2, group_sizes=(2, 1), exact_group_mask=0b10)])
def test_rules_on_trees(rule):
    wl = synth.Workload("tree_rules", SMALL64, 0, 24, SMALL64.bin_base, batch=4, K=7, draft=("geometric", 0.5), seed=31)
    run_tree_case(wl, 3, rule, p_geo=0.6)


@pytest.mark.parametrize("n_bins,sizes,mask", [(48, (300,), 0), (528, (1, 2, 1, 3, 1, 1, 2, 1), 0b10010001), (256, (5, 257), 0b1)])
def test_bin_counts_and_patterns_of_the_acceptance(n_bins, sizes, mask):
    """Fewer bins than a slice of a row and more than one round of four, not a multiple of a wave; a pattern longer than any chain, one
    of eight groups, one whose last group never ends.  (The oracle's decisions: whole numbers.)"""
    sh = synth.ModelShape(n_layers=2, d_model=256, n_heads=4, head_dim=64, d_ffn=688, vocab=1024, n_bins=n_bins)
    wl = synth.Workload("tree_bins_%d" % n_bins, sh, 0, 24, sh.bin_base, batch=2, K=14, draft=("geometric", 0.5), seed=n_bins)
    run_tree_case(wl, 3, oracle.AcceptRule(6, 40, group_sizes=sizes, exact_group_mask=mask), p_geo=0.6)


def test_one_chain_tree_equals_the_linear_step_on_the_gpu():
    from gpu_harness import run_gpu_step, run_gpu_tree_step
    _need_gpu()
    wl = synth.Workload("tree_lin", SMALL64, 0, 30, SMALL64.bin_base, batch=2, K=7, seed=9)
    weights = synth.make_weights(wl.shape, wl.seed)
    cap = 44
    k0, v0, f0 = zip(*[synth.make_prefix_kv_direct(wl, e, cap) for e in range(2)])
    kb, vb = np.stack(k0, axis=1), np.stack(v0, axis=1)
    drafts = (wl.shape.bin_base + synth.make_drafts_uniform(wl)).astype(np.int32)
    parent = np.tile(np.arange(-1, 6, dtype=np.int32), (2, 1))
    rule = oracle.AcceptRule(15, 30)
    lin = run_gpu_step(wl.shape, weights, kb, vb, [30, 30], list(f0), drafts, rule, None, path=4)
    tree = run_gpu_tree_step(wl.shape, weights, kb, vb, [30, 30], list(f0), drafts, parent, rule, None, path=4)
    for k in ("accepted_len", "next_token", "target_bins", "bin_logits", "k_cache", "v_cache"):
        assert np.array_equal(lin[k], tree[k]), k
    for b in range(2):
        n = int(tree["accepted_len"][b])
        assert tree["accepted_path"][b, :n].tolist() == list(range(n))


def test_tree_step_argument_errors():
    from paper_2603_17573_amd import DeviceModel, Verifier, make_accept_desc, binding as B
    _need_gpu()
    wl = synth.Workload("tree_err", SMALL64, 0, 8, 1024, batch=2, K=7, seed=1)
    dm = DeviceModel(wl.shape, synth.make_weights(wl.shape, 1))
    ver = Verifier(dm, max_batch=2, max_k=16, kv_capacity=40)
    kc, vc = ver.new_cache(2)
    z = torch.zeros(2, dtype=torch.int32, device="cuda")
    tok = torch.full((2, 16), wl.shape.bin_base, dtype=torch.int32, device="cuda")
    par = torch.arange(-1, 15, dtype=torch.int32, device="cuda").repeat(2, 1).contiguous()
    acc = torch.full((2,), -7, dtype=torch.int32, device="cuda")
    nxt = torch.full((2,), -7, dtype=torch.int32, device="cuda")
    kv = B.heisd_kv_desc(kc.data_ptr(), vc.data_ptr(), z.data_ptr(), z.data_ptr())
    ok = make_accept_desc(2, 6)

    def call(T=16, batch=2, accept=ok, parent=par.data_ptr(), out=acc.data_ptr()):
        return B.heisd_verify_tree_step(ver.ctx, kv, tok.data_ptr(), parent, T, batch, accept, None, out,
                                        nxt.data_ptr(), None, None, None, None)

    assert call(T=17) == B.HEISD_EINVAL and call(T=0) == B.HEISD_EINVAL and call(batch=3) == B.HEISD_EINVAL
    assert call(parent=None) == B.HEISD_EINVAL and call(out=None) == B.HEISD_EINVAL
    assert call(accept=make_accept_desc(2, 6, mode=3)) == B.HEISD_EINVAL
    assert B.heisd_verify_set_path(ver.ctx, B.HEISD_PATH_FAST) == 0
    assert call() == B.HEISD_EUNSUPPORTED
    assert B.heisd_verify_set_path(ver.ctx, B.HEISD_PATH_AUTO) == 0
    torch.cuda.synchronize()
    assert acc.tolist() == [-7, -7]
    assert call() == B.HEISD_OK                    # accepted_path NULL: the library keeps it in its workspace
    torch.cuda.synchronize()
    assert all(0 <= v <= 16 for v in acc.tolist())
    ver.close()


@pytest.mark.parametrize("shape,B,K,R", [(MID, 65, 7, 1), (SMALL64, 70, 3, 2), (MID, 33, 6, 2), (SMALL64, 35, 9, 1)])
def test_many_episodes_around_a_tile(shape, B, K, R):
    """More workgroups than compute units, trees of at most 8 tokens (one block of queries per episode) and of more, prefixes on both
    sides of a 32-key tile, skipped episodes."""
    wl = synth.Workload("tree_many_%d_%d" % (B, K), shape, 0, 33, shape.bin_base, batch=B, K=K, draft=("geometric", 0.5), seed=B)
    skip = (np.arange(B) % 7 == 3).astype(np.uint8)
    got, ref, stats, tokens, parent = run_tree_case(wl, R, oracle.AcceptRule(15, 30), p_geo=0.6, skip=skip, path=4,
                                                    plen_override=33 - np.arange(B) % 4)
    assert (tokens.shape[1] <= 8) == (R * K <= 8)
