"""GPU parity: sx_draft_tree (Alg. 2, createDraftTree on the device) against the oracle's heap version."""
import numpy as np
import pytest
import torch

import oracle
import workloads as wl
from helpers import dev, to_dev, weights_to, weights_np

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sx():
    import paper_2406_02532_amd as m
    return m


@pytest.fixture(scope="module")
def draft():
    """A small fp32 draft model with sharp next-token distributions and a cached prefix."""
    cfg = wl.ModelCfg(2, 128, 4, 2, 32, 256, 300, dtype="fp32")
    w = wl.gen_weights(cfg, seed=61)
    w = dict(w, lm_head=w["lm_head"] * 12.0, embed=w["embed"] * 20.0)
    wn = weights_np(w)
    prefix = wl.gen_tokens(24, cfg.vocab, seed=62)
    _, pk, pv = oracle.path_forward(cfg, wn, None, None, prefix, return_kv=True)
    return cfg, w, wn, pk, pv


def _safe(ref, cfg, wn, pk, pv):
    """No two scores that decide an order sit within 1e-4 of each other: the tree's scores and siblings."""
    c = np.sort(ref["cum_logp"].astype(np.float64))
    return len(c) < 2 or np.min(np.diff(c)) > 1e-4


@pytest.mark.parametrize("K,D,B,k", [(12, 6, 4, 3), (40, 8, 8, 4), (30, 4, 16, 5), (64, 10, 16, 8), (9, 30, 1, 6)])
def test_draft_tree_equals_oracle(sx, draft, K, D, B, k):
    cfg, w, wn, pk, pv = draft
    P = pk.shape[1]
    mw = sx.ModelWeights(cfg, weights_to(w, dev()))
    pkd, pvd = to_dev(torch.as_tensor(pk), torch.float32), to_dev(torch.as_tensor(pv), torch.float32)
    checked = 0
    for root in (5, 77, 123, 250):
        ref = oracle.create_draft_tree(cfg, wn, pk, pv, root, K=K, D=D, B=B, k=k)
        if not _safe(ref, cfg, wn, pk, pv):
            continue
        toks, par, cum, n, ws = sx.draft_tree(mw, pkd, pvd, P, torch.tensor([root], dtype=torch.int32, device=dev()),
                                              K, D, B, k)
        torch.cuda.synchronize()
        assert sx.check_status(ws) == 0
        n = int(n.item())
        assert n == len(ref["tokens"])
        assert toks[:n].cpu().tolist() == ref["tokens"].tolist()
        assert par[:n].cpu().tolist() == ref["parent"].tolist()
        np.testing.assert_allclose(cum[:n].cpu().numpy(), ref["cum_logp"], atol=2e-4)
        checked += 1
    assert checked >= 2


@pytest.mark.parametrize("K,D,B,k", [(40, 3, 32, 8), (40, 3, 43, 6), (250, 6, 50, 5), (260, 6, 64, 4), (40, 3, 32, 33), (1050, 4, 300, 4)])
def test_draft_tree_on_both_sides_of_256_candidates(sx, draft, K, D, B, k):
    """Up to 256 candidates, queue entries and slots are ordered by counting, the picks by the step that pops them; more go
    through the general selection, a sorting network and a bit search.  Near-equal scores may change places: the scores of
    the tree, every node's against its parent's, and the tree itself where no two scores are close."""
    cfg, w, wn, pk, pv = draft
    mw = sx.ModelWeights(cfg, weights_to(w, dev()))
    pkd, pvd = to_dev(torch.as_tensor(pk), torch.float32), to_dev(torch.as_tensor(pv), torch.float32)
    ref = oracle.create_draft_tree(cfg, wn, pk, pv, 77, K=K, D=D, B=B, k=k)
    toks, par, cum, n, ws = sx.draft_tree(mw, pkd, pvd, pk.shape[1], torch.tensor([77], dtype=torch.int32, device=dev()), K, D, B, k)
    torch.cuda.synchronize()
    assert sx.check_status(ws) == 0
    n = int(n.item())
    assert n == len(ref["tokens"])
    toks, par, cum = toks[:n].cpu().numpy(), par[:n].cpu().numpy(), cum[:n].cpu().numpy()
    np.testing.assert_allclose(np.sort(cum), np.sort(ref["cum_logp"]), atol=2e-4)
    assert par[0] == -1 and all(0 <= par[i] < i and cum[i] <= cum[par[i]] for i in range(1, n))
    pairs = list(zip(par.tolist(), toks.tolist()))
    assert len(set(pairs)) == n
    if _safe(ref, cfg, wn, pk, pv):
        assert toks.tolist() == ref["tokens"].tolist() and par.tolist() == ref["parent"].tolist()


def test_draft_tree_feeds_verify_tree(sx, draft):
    """The tree that comes out is a valid input of the verification forward (topological order, one root)."""
    cfg, w, wn, pk, pv = draft
    P = pk.shape[1]
    mw = sx.ModelWeights(cfg, weights_to(w, dev()))
    pkd, pvd = to_dev(torch.as_tensor(pk), torch.float32), to_dev(torch.as_tensor(pv), torch.float32)
    toks, par, cum, n, ws = sx.draft_tree(mw, pkd, pvd, P, torch.tensor([9], dtype=torch.int32, device=dev()), 48, 8, 16, 6)
    torch.cuda.synchronize()
    n = int(n.item())
    assert 1 <= n <= 48
    logits, ws2 = sx.verify_tree(mw, pkd, pvd, toks[:n].contiguous(), par[:n].contiguous())
    torch.cuda.synchronize()
    assert sx.check_status(ws2) == 0
    ref = oracle.verify_tree(cfg, wn, pk, pv, toks[:n].cpu().numpy(), par[:n].cpu().numpy())["logits"]
    assert np.abs(logits.cpu().double().numpy() - ref).max() <= 1e-4


def test_draft_tree_rejects_unsupported_shapes(sx, draft):
    cfg, w, wn, pk, pv = draft
    mw = sx.ModelWeights(cfg, weights_to(w, dev()))
    root = torch.tensor([1], dtype=torch.int32, device=dev())
    with pytest.raises(sx.SxError):
        sx.draft_tree(mw, None, None, 0, root, 10, 20000, 1, 4)          # D * B over the limit
    with pytest.raises(sx.SxError):
        sx.draft_tree(mw, None, None, 0, root, 0, 4, 4, 4)               # K < 1


@pytest.mark.parametrize("draft_kind", ["unrelated", "self"])
def test_speculative_generation_end_to_end_equals_sequential_sampling(sx, draft_kind):
    """The whole of Alg. 1 with Alg. 2 inside, every step on the device: each round the draft model builds a tree
    (sx_draft_tree), the target verifies it, walks it and commits the accepted nodes (sx_specexec_round), and the
    draft model's own cache is brought up to date.  Sect. 4.1: the emitted tokens are exactly what token-by-token
    sampling from the TARGET model gives with the same seed, whatever the draft model proposes."""
    tcfg = wl.ModelCfg(2, 256, 4, 4, 64, 688, 1024, dtype="fp32")
    dcfg = wl.ModelCfg(1, 128, 4, 2, 32, 256, 1024, dtype="fp32")
    tw = wl.gen_weights(tcfg, seed=71)
    tw = dict(tw, lm_head=tw["lm_head"] * 20.0)
    # "unrelated": another random model, whose guesses the target almost never accepts (one token per round);
    # "self": the target drafts for itself, so most rounds accept several tokens
    if draft_kind == "self":
        dcfg, dw = tcfg, tw
    else:
        dw = wl.gen_weights(dcfg, seed=72)
        dw = dict(dw, lm_head=dw["lm_head"] * 10.0)
    twn, dwn = weights_np(tw), weights_np(dw)
    prompt = [int(t) for t in wl.gen_tokens(12, tcfg.vocab, seed=73)]
    P0 = len(prompt) - 1
    _, tpk, tpv = oracle.path_forward(tcfg, twn, None, None, prompt[:-1], return_kv=True)
    _, dpk, dpv = oracle.path_forward(dcfg, dwn, None, None, prompt[:-1], return_kv=True)
    tmw, dmw = sx.ModelWeights(tcfg, weights_to(tw, dev())), sx.ModelWeights(dcfg, weights_to(dw, dev()))
    rounds, K, D, B, k = 4, 24, 5, 8, 4
    cap = P0 + rounds * K
    checked, accepted = 0, 0
    for s in range(40):
        if checked >= 3:
            break
        truth = oracle.sequential_sample(tcfg, twn, tpk, tpv, prompt[-1], rounds * 4 + 2, 0.6, 0.9, seed=s, pos0=P0)
        seq, safe = [prompt[-1]], True
        for x in truth:                                                # every decision safely away from a tie
            lg = oracle.path_forward(tcfg, twn, tpk, tpv, seq)
            _, m = oracle.sample_token(lg, 0.6, 0.9, oracle.uniform01(s, P0 + len(seq)))
            safe &= min(m["m_p"], m["m_u"]) > 1e-3
            seq.append(x)
        if not safe:
            continue

        def cache(cfg, pk, pv):
            ck = torch.zeros((cfg.n_layers, cap, cfg.n_kv_heads, cfg.head_dim), dtype=torch.float32, device=dev())
            cv = torch.zeros_like(ck)
            ck[:, :P0] = to_dev(torch.as_tensor(pk), torch.float32)
            cv[:, :P0] = to_dev(torch.as_tensor(pv), torch.float32)
            return ck, cv
        tck, tcv = cache(tcfg, tpk, tpv)
        dck, dcv = cache(dcfg, dpk, dpv)
        buf = sx.RoundBuffers(tmw, cap, K)
        P, root, emitted = P0, torch.tensor([prompt[-1]], dtype=torch.int32, device=dev()), []
        for rd in range(rounds):
            toks, par, cum, n, ws = sx.draft_tree(dmw, dck, dcv, P, root, K, D, B, k)
            torch.cuda.synchronize()
            assert sx.check_status(ws) == 0
            nt = int(n.item())
            tree_t, tree_p = toks[:nt].contiguous(), par[:nt].contiguous()
            sx.specexec_round(tmw, tck, tcv, P, tree_t, tree_p, 0.6, 0.9, s, buf)
            torch.cuda.synchronize()
            assert sx.check_status(buf.workspace) == 0
            na = int(buf.n.item())
            out = buf.tokens[:na].cpu().tolist()
            # the draft model's cache takes the same accepted tokens: a chain forward, then the same commit
            chain = torch.tensor([int(root.item())] + out[:-1], dtype=torch.int32, device=dev())
            cpar = torch.arange(-1, na - 1, dtype=torch.int32, device=dev())
            dk = torch.zeros((dcfg.n_layers, na, dcfg.n_kv_heads, dcfg.head_dim), dtype=torch.float32, device=dev())
            dv = torch.zeros_like(dk)
            sx.verify_tree(dmw, dck, dcv, chain, cpar, tree_k_out=dk, tree_v_out=dv, P=P)
            sx.commit_kv(dcfg, dck, dcv, P, dk, dv, torch.arange(na, dtype=torch.int32, device=dev()),
                         torch.tensor([na], dtype=torch.int32, device=dev()))
            emitted += out
            P += na
            root = torch.tensor([out[-1]], dtype=torch.int32, device=dev())
        if len(emitted) > len(truth):        # more accepted than the margin check covered: compare what it covers
            emitted = emitted[:len(truth)]
        assert emitted == truth[:len(emitted)] and len(emitted) >= rounds
        accepted += len(emitted) - rounds
        checked += 1
    assert checked >= 3
    if draft_kind == "self":
        assert accepted >= 3                 # drafting with the target itself must get draft tokens accepted


def test_draft_tree_bf16_model_close_to_oracle(sx):
    """The MFMA path of the draft loop (narrow-tile GEMMs with K cut in parts, small attention tiles, rotation in the
    QKV product's epilogue, growing tree K/V in bf16) against the oracle evaluating the same bf16 model.  Two bf16
    evaluations differ by rounding flips (a few 1e-3 in log-probability), which can swap candidates whose scores
    nearly tie; so: scores of the nodes both trees contain agree to 0.05, and at least 90% of the nodes coincide."""
    cfg = wl.ModelCfg(2, 512, 4, 2, 128, 1408, 2000, dtype="bf16")
    w = wl.gen_weights(cfg, seed=81)
    w = dict(w, lm_head=(w["lm_head"].float() * 12.0).to(torch.bfloat16), embed=(w["embed"].float() * 20.0).to(torch.bfloat16))
    P = 40
    pk, pv = wl.gen_prefix_kv(cfg, P, seed=82)
    mw = sx.ModelWeights(cfg, weights_to(w, dev()))
    K, D, B, k = 60, 6, 32, 6
    ref = oracle.create_draft_tree(cfg, w, pk, pv, 11, K=K, D=D, B=B, k=k, act_round="bf16")
    toks, par, cum, n, ws = sx.draft_tree(mw, pk.to(dev()), pv.to(dev()), P, torch.tensor([11], dtype=torch.int32, device=dev()),
                                          K, D, B, k)
    torch.cuda.synchronize()
    assert sx.check_status(ws) == 0
    n = int(n.item())
    got = dict(tokens=toks[:n].cpu().numpy(), parent=par[:n].cpu().numpy(), cum_logp=cum[:n].cpu().numpy())

    def paths(t):
        out = {}
        for i in range(len(t["tokens"])):
            p, j = [], i
            while j >= 0:
                p.append(int(t["tokens"][j]))
                j = int(t["parent"][j])
            out[tuple(reversed(p))] = float(t["cum_logp"][i])
        return out
    a, b = paths(ref), paths(got)
    common = set(a) & set(b)
    assert n == len(ref["tokens"]) == K
    assert len(common) >= 0.9 * K, (len(common), K)
    assert max(abs(a[p] - b[p]) for p in common) <= 0.05
    assert all(-1 <= got["parent"][i] < i for i in range(n))


def test_draft_tree_degenerate_budgets(sx, draft):
    """K = 1 (the root alone), one iteration, no cached prefix: the smallest trees the loop can return."""
    cfg, w, wn, pk, pv = draft
    mw = sx.ModelWeights(cfg, weights_to(w, dev()))
    root = torch.tensor([42], dtype=torch.int32, device=dev())
    toks, par, cum, n, ws = sx.draft_tree(mw, None, None, 0, root, 1, 3, 4, 2)          # K = 1
    torch.cuda.synchronize()
    assert sx.check_status(ws) == 0 and int(n.item()) == 1
    assert toks[:1].cpu().tolist() == [42] and par[:1].cpu().tolist() == [-1] and float(cum[0]) == 0.0
    ref = oracle.create_draft_tree(cfg, wn, np.zeros((cfg.n_layers, 0, cfg.n_kv_heads, cfg.head_dim)),
                                   np.zeros((cfg.n_layers, 0, cfg.n_kv_heads, cfg.head_dim)), 42, K=6, D=1, B=8, k=3)
    toks, par, cum, n, ws = sx.draft_tree(mw, None, None, 0, root, 6, 1, 8, 3)          # D = 1: only the root is expanded
    torch.cuda.synchronize()
    assert int(n.item()) == len(ref["tokens"]) == 1
    ref = oracle.create_draft_tree(cfg, wn, np.zeros((cfg.n_layers, 0, cfg.n_kv_heads, cfg.head_dim)),
                                   np.zeros((cfg.n_layers, 0, cfg.n_kv_heads, cfg.head_dim)), 42, K=5, D=2, B=8, k=3)
    toks, par, cum, n, ws = sx.draft_tree(mw, None, None, 0, root, 5, 2, 8, 3)          # root + its 3 best children
    torch.cuda.synchronize()
    n = int(n.item())
    assert n == len(ref["tokens"]) == 4
    assert toks[:n].cpu().tolist() == ref["tokens"].tolist() and par[:n].cpu().tolist() == ref["parent"].tolist()


def test_draft_tree_recorded_in_a_graph_replays_the_eager_result(sx):
    """sx_draft_tree only enqueues kernels (no allocation, no host synchronisation, no memset nodes), so a caller
    may record it into a HIP graph and replay it, which removes the gaps between its thousands of short launches.
    A bf16 draft model (the narrow GEMMs with K cut among workgroups, whose counters must be left clean for the
    next replay): three replays, each after eager work and a synchronisation, each equal to the eager call."""
    cfg = wl.ModelCfg(3, 512, 8, 2, 128, 1408, 2000, dtype="bf16")
    K, D, B, k, P = 96, 6, 32, 6, 80
    w = wl.gen_weights(cfg, seed=71, device=dev())
    w["lm_head"] = (w["lm_head"].float() * 10).to(torch.bfloat16)
    mw = sx.ModelWeights(cfg, w)
    pk, pv = wl.gen_prefix_kv(cfg, P, seed=72, device=dev())
    root = torch.tensor([41], dtype=torch.int32, device=dev())
    toks, par, cum, n, ws = sx.draft_tree(mw, pk, pv, P, root, K, D, B, k)
    torch.cuda.synchronize()
    assert sx.check_status(ws) == 0 and int(n.item()) > 8
    eager = [t.clone() for t in (toks, par, cum, n)]
    outs = tuple(torch.zeros_like(t) for t in eager)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        sx.draft_tree(mw, pk, pv, P, root, K, D, B, k, workspace=ws, out=outs)
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=side):
        sx.draft_tree(mw, pk, pv, P, root, K, D, B, k, workspace=ws, out=outs)
    for rep in range(3):
        for t in outs:
            t.zero_()                                    # eager work between the replays
        junk = torch.randn(1 << 20, device=dev()).sum()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert sx.check_status(ws) == 0
        for a, b in zip(outs, eager):
            assert torch.equal(a, b), f"replay {rep} differs from the eager call"
    del junk


@pytest.mark.parametrize("k", [4, 32, 56])
def test_draft_tree_without_room_for_shared_rows(sx, k):
    """A vocabulary whose rows the expansion shares among workgroups: a workspace without the room for that is taken, down to
    the last byte of the rest, and gives the same tree."""
    cfg = wl.ModelCfg(1, 128, 4, 2, 32, 256, 50257, dtype="fp32")
    w = wl.gen_weights(cfg, seed=71)
    mw = sx.ModelWeights(cfg, weights_to(dict(w, lm_head=w["lm_head"] * 12.0, embed=w["embed"] * 20.0), dev()))
    P, K, D, B = 24, 200, 3, 64
    kv = lambda key: wl.hash_normal(key, (1, P, 2, 32), device=dev())  # noqa: E731
    root = torch.tensor([7], dtype=torch.int32, device=dev())
    full = sx.draft_tree(mw, kv(1), kv(2), P, root, K, D, B, k)
    q = sx.lib.sx_expand_topk_workspace
    least = full[4].numel() - (q(B, cfg.vocab, k, K) - q(B, 1, k, K))
    assert least < full[4].numel()
    got = sx.draft_tree(mw, kv(1), kv(2), P, root, K, D, B, k, workspace=torch.empty(least, dtype=torch.uint8, device=dev()))
    n = int(full[3].item())
    assert n == int(got[3].item()) > 1
    for i in range(2):
        assert torch.equal(full[i][:n], got[i][:n])
    np.testing.assert_allclose(got[2][:n].cpu().numpy(), full[2][:n].cpu().numpy(), rtol=0, atol=1e-4)
    with pytest.raises(sx.SxError) as e:
        sx.draft_tree(mw, kv(1), kv(2), P, root, K, D, B, k, workspace=torch.empty(least - 256, dtype=torch.uint8, device=dev()))
    assert e.value.code == -3
