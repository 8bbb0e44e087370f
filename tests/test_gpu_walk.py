"""GPU parity: sx_accept_walk against the oracle's walk (Alg. 1, main loop) -- paths and sampled
tokens bit-exact on fixtures whose decision margins are safe for fp32."""
import numpy as np
import pytest
import torch

import oracle
import workloads as wl
from helpers import dev, to_dev

pytestmark = pytest.mark.gpu

MARGIN = 1e-4   # decisions closer than this (in probability mass) may legitimately flip in fp32


@pytest.fixture(scope="module")
def sx():
    import paper_2406_02532_amd as m
    return m


def _walk(sx, logits_d, tok_d, par_d, t, top_p, seed, pos0):
    path, toks, n, ws = sx.accept_walk(logits_d, tok_d, par_d, t, top_p, seed, pos0)
    torch.cuda.synchronize()
    n = int(n.item())
    return path[:n].cpu().tolist(), toks[:n].cpu().tolist(), ws


def _safe(ref):
    return all(min(m["m_p"], m["m_u"], m["m_top"]) > MARGIN for m in ref["margins"])


@pytest.mark.parametrize("V,T", [(1024, 64), (1000, 40), (8000, 64), (32000, 256), (32768, 32), (50000, 32), (131072, 16)])
@pytest.mark.parametrize("t,top_p", [(0.6, 0.9), (0.0, 1.0), (1.0, 1.0), (0.3, 0.5)])
def test_walk_matches_oracle(sx, V, T, t, top_p):
    """Sharp (LLM-like) rows: every decision has a wide margin, so paths and tokens are bit-exact."""
    tok, par, _ = wl.gen_best_first_tree(T, 4, V, seed=V + T, max_depth=12)
    logits = wl.gen_crafted_logits(tok, par, V, seed=V + 1, boost=9.0, sharp=True)
    ld, td, pd = to_dev(logits), to_dev(tok), to_dev(par)
    checked, longest = 0, 0
    for seed in range(16):
        ref = oracle.accept_walk(logits, tok, par, t, top_p, seed=seed, pos0=17)
        if not _safe(ref):
            continue
        path, toks, _ = _walk(sx, ld, td, pd, t, top_p, seed, 17)
        assert path == ref["path"], (seed, path, ref["path"])
        assert toks == ref["tokens"]
        checked += 1
        longest = max(longest, len(path))
    assert checked >= 8
    if t <= 0.6:
        assert longest >= 2          # sharp distributions: the walk does go down the tree


@pytest.mark.parametrize("V", [1024, 32000, 128256])
def test_walk_on_flat_rows_is_valid(sx, V):
    """Flat N(0,1) rows: thousands of near-equal probabilities, so nucleus edge and CDF edges are
    closer than fp32 can tell apart.  Each step must then be *a* correct draw: the token the
    oracle returns for some (top_p, u) within 1e-4 of the nominal values; steps whose margins
    are safe must match exactly.  Comparison stops at the first legitimately different token."""
    T = 48
    tok, par, _ = wl.gen_best_first_tree(T, 4, V, seed=V, max_depth=8)
    logits = wl.gen_crafted_logits(tok, par, V, seed=V + 2, boost=9.0)
    ld, td, pd = to_dev(logits), to_dev(tok), to_dev(par)
    depth = oracle.tree_depths(par)
    steps = 0
    for seed in range(10):
        path, toks, _ = _walk(sx, ld, td, pd, 0.6, 0.9, seed, 5)
        ref = oracle.accept_walk(logits, tok, par, 0.6, 0.9, seed=seed, pos0=5)
        assert path[0] == 0
        for s, (node, g) in enumerate(zip(path, toks)):
            assert node == ref["path"][s]
            m = ref["margins"][s]
            if g == ref["tokens"][s]:
                steps += 1
                continue
            assert min(m["m_p"], m["m_u"]) <= MARGIN, "safe step but different token"
            u = oracle.uniform01(seed, 5 + int(depth[node]) + 1)
            alts = {oracle.sample_token(logits[node], 0.6, 0.9 + dp, min(max(u + du, 0.0), 1 - 2 ** -24))[0]
                    for dp in (-1e-4, 0.0, 1e-4) for du in (-1e-4, -3e-5, 0.0, 3e-5, 1e-4)}
            assert g in alts
            break
    assert steps >= 10


def test_nucleus_with_tied_probabilities(sx):
    """Equal logits at the nucleus boundary: ties enter in id order (hand-checkable case)."""
    V = 1024
    logits = np.full((1, V), -30.0, dtype=np.float32)
    logits[0, [5, 100, 200, 900]] = [np.log(0.5), np.log(0.2), np.log(0.2), np.log(0.1)]
    tok, par = np.array([3], np.int32), np.array([-1], np.int32)
    ld, td, pd = to_dev(logits), to_dev(tok), to_dev(par)
    for seed in range(40):
        ref = oracle.accept_walk(logits, tok, par, 1.0, 0.6, seed=seed, pos0=0)
        if ref["margins"][0]["m_u"] < MARGIN:
            continue
        path, toks, _ = _walk(sx, ld, td, pd, 1.0, 0.6, seed, 0)
        assert toks == ref["tokens"] and toks[0] in (5, 100)      # token 200 ties with 100 but has the higher id


@pytest.mark.parametrize("V,top_p", [(1023, 0.9), (4097, 0.75), (32767, 0.9), (40001, 0.66), (128256, 1.0)])
@pytest.mark.parametrize("tied", [False, True])
def test_walk_with_any_number_of_candidates(sx, V, top_p, tied):
    """Rows whose nucleus comes from c likely tokens over a floor too low to matter, c on both sides of what the kernel
    finishes in one wave (64), in its list (1024) and with the whole row; rows that are no multiple of four long."""
    r = np.random.default_rng(V)
    checked = 0
    for c in (1, 3, 63, 64, 65, 200, 1000, 1024, 1025, 3000):
        if c > V:
            continue
        lg = np.full((1, V), -40.0, np.float32)
        ids = r.choice(V, size=c, replace=False)
        lg[0, ids] = 1.0 if tied else r.uniform(0.0, 3.0, size=c).astype(np.float32)
        lg[0, V - 1] = lg[0, ids[0]]
        tok, par = np.array([3], np.int32), np.array([-1], np.int32)
        ld, td, pd = to_dev(lg), to_dev(tok), to_dev(par)
        qd = to_dev(np.full((1, V), 1.0 / V, np.float32))
        for seed in range(6):
            ref = oracle.accept_walk(lg, tok, par, 0.8, top_p, seed=seed, pos0=9)
            m = ref["margins"][0]
            if min(m["m_p"], m["m_u"]) > 1e-5:      # sums of at most 3000 terms: fp32 terms are good to 3e-7 of the mass
                path, toks, _ = _walk(sx, ld, td, pd, 0.8, top_p, seed, 9)
                assert path == [0] and toks == ref["tokens"], (c, seed)
                checked += 1
            ref = oracle.specinfer_walk(lg, np.full((1, V), 1.0 / V), tok, par, 0.8, top_p, seed=seed, pos0=9)
            if min(ref["margins"][0]["m_acc"], ref["margins"][0]["m_u"]) > 1e-5 and m["m_p"] > 1e-5:
                _, toks, n, _ = sx.accept_walk(ld, td, pd, 0.8, top_p, seed, 9, draft_probs=qd)
                torch.cuda.synchronize()
                assert int(n.item()) == 1 and int(toks[0].item()) == ref["tokens"][0], (c, seed)
                checked += 1
    assert checked >= 12


@pytest.mark.parametrize("V", [1000, 4095, 32000, 32768, 40001, 131072])
@pytest.mark.parametrize("top_p", [0.7, 1.0])
def test_walk_on_masked_rows(sx, V, top_p):
    """Rows of which all but c tokens are masked out (-inf): only those can be drawn, by both walks, with c on both sides
    of what the kernel finishes in one wave, in its list and over the whole row; ids at both ends of the row and of the
    256-id blocks of its sums.  A row with nothing left gives token 0."""
    r = np.random.default_rng(V)
    tok, par = np.array([3], np.int32), np.array([-1], np.int32)
    td, pd = to_dev(tok), to_dev(par)
    qd = to_dev(np.full((1, V), 1.0 / V, np.float32))
    checked = 0
    for c in (1, 2, 70, 1024, 1025, 2000, V):
        if c > V:
            continue
        lg = np.full((1, V), -np.inf, np.float32)
        ends = np.array([0, V - 1, 255, 256, V - 2, V // 256 * 256 - 1])[:c]
        ids = np.concatenate([ends, r.permutation(np.setdiff1d(np.arange(V), ends))[:c - len(ends)]])
        lg[0, ids] = r.normal(0.0, 2.0, size=len(ids)).astype(np.float32) + 20.0
        ld = to_dev(lg)
        for seed in range(8):
            ref = oracle.accept_walk(lg, tok, par, 0.9, top_p, seed=seed, pos0=9)
            m = ref["margins"][0]
            # the exponentials are good to 1e-6 and independent: sums over the row to a few 1e-8 of the mass
            if min(m["m_p"], m["m_u"]) > 2e-7:
                assert _walk(sx, ld, td, pd, 0.9, top_p, seed, 9)[1] == ref["tokens"], (c, seed)
                checked += 1
            ref = oracle.specinfer_walk(lg, np.full((1, V), 1.0 / V), tok, par, 0.9, top_p, seed=seed, pos0=9)
            if ref["margins"][0]["m_u"] > 2e-7 and m["m_p"] > 2e-7:
                _, toks, n, _ = sx.accept_walk(ld, td, pd, 0.9, top_p, seed, 9, draft_probs=qd)
                torch.cuda.synchronize()
                assert int(n.item()) == 1 and int(toks[0].item()) == ref["tokens"][0], (c, seed)
                checked += 1
    assert checked >= 60
    ld = to_dev(np.full((1, V), -np.inf, np.float32))
    assert _walk(sx, ld, td, pd, 0.9, top_p, 1, 9)[1] == [0]
    assert _walk(sx, ld, td, pd, 0.0, top_p, 1, 9)[1] == [0]


@pytest.mark.parametrize("M,t,V,above", [(-100.0, 1e-3, 32000, False), (37.0, 2e-4, 32000, True), (100.0, 1e-3, 50001, True)])
def test_walk_on_rows_with_an_offset(sx, M, t, V, above):
    """A row far from zero and sharpened by a low temperature, whose many small probabilities (a tenth of the mass, each
    too small for the nucleus) decide whether the nucleus is one token or two: their sum must come from the differences
    to the maximum.  (From logits and maximum scaled apart its relative error is |M| / t * 1e-7, ten times the margin.)"""
    f = np.float32
    r = np.random.default_rng(0)
    e = lambda x: np.exp((np.float64(x) - np.float64(f(M))) / np.float64(f(t)))  # noqa: E731
    grid = [f(M)]
    while e(grid[-1]) > 2e-5:
        grid.append(np.nextafter(grid[-1], f(-np.inf)))
    weights = np.array([e(x) for x in grid])
    lg = np.full((1, V), f(M - t * 12.8), f)
    ids = r.permutation(V)
    lg[0, ids[0]] = M                                    # weight 1; top_p 0.5 asks whether the others weigh more than 1
    left = 1.0 - e(lg[0, ids[1]]) * (V - 61) + (3e-4 if above else -3e-4)
    k = 1
    while k < 61 and left > 2e-5:
        j = int(np.argmax(weights <= min(left, 0.3 - 0.01 * min(k, 20))))   # no two alike
        lg[0, ids[k]] = grid[j]
        left -= weights[j]
        k += 1
    tok, par = np.array([3], np.int32), np.array([-1], np.int32)
    ld, td, pd = to_dev(lg), to_dev(tok), to_dev(par)
    checked = 0
    for seed in range(40):
        ref = oracle.accept_walk(lg, tok, par, t, 0.5, seed=seed, pos0=2)
        m = ref["margins"][0]
        assert 2e-5 < m["m_p"] < 2e-4
        if m["m_u"] > MARGIN:
            assert _walk(sx, ld, td, pd, t, 0.5, seed, 2)[1] == ref["tokens"], seed
            checked += 1
    assert checked >= 30


def test_duplicate_siblings_and_single_node(sx):
    tok = np.array([5, 3, 3, 9], np.int32)
    par = np.array([-1, 0, 0, 1], np.int32)
    logits = np.full((4, 16), -20.0, dtype=np.float32)
    logits[0, 3] = logits[1, 9] = logits[2, 1] = logits[3, 2] = 0.0
    path, toks, _ = _walk(sx, to_dev(logits), to_dev(tok), to_dev(par), 0.0, 1.0, 1, 0)
    assert path == [0, 1, 3] and toks == [3, 9, 2]
    path, toks, _ = _walk(sx, to_dev(logits[:1]), to_dev(tok[:1]), to_dev(par[:1]), 0.6, 0.9, 1, 0)
    assert path == [0] and toks == [3]


def test_chain_is_walked_to_its_end(sx):
    """A chain whose every row points at the next node: the walk visits all T nodes (its maximum)."""
    T, V = 50, 300
    tok, par = wl.gen_chain_tree(T, V, seed=4)
    logits = np.full((T, V), -25.0, dtype=np.float32)
    for i in range(T - 1):
        logits[i, tok[i + 1]] = 0.0
    logits[T - 1, 7] = 0.0
    path, toks, _ = _walk(sx, to_dev(logits), to_dev(tok), to_dev(par), 0.6, 0.9, 3, 100)
    assert path == list(range(T)) and toks == tok[1:].tolist() + [7]


def test_root_must_be_node_zero(sx):
    tok = np.array([1, 2], np.int32)
    par = np.array([0, -1], np.int32)        # node 0 is not a root
    logits = np.zeros((2, 8), np.float32)
    _, _, ws = _walk(sx, to_dev(logits), to_dev(tok), to_dev(par), 0.0, 1.0, 0, 0)
    assert sx.check_status(ws) == -6
    par = np.array([-1, 0], np.int32)
    _, _, ws = _walk(sx, to_dev(logits), to_dev(tok), to_dev(par), 0.0, 1.0, 0, 0)
    assert sx.check_status(ws) == 0


def test_plain_categorical_frequencies(sx):
    """t=1, top_p=1 on a 6-token row over many seeds: chi-square against the exact probabilities."""
    p = np.array([0.02, 0.4, 0.08, 0.25, 0.05, 0.2])
    logits = np.log(p).astype(np.float32)[None, :]
    tok, par = np.array([0], np.int32), np.array([-1], np.int32)
    ld, td, pd = to_dev(logits), to_dev(tok), to_dev(par)
    n = 4000
    outs = [sx.accept_walk(ld, td, pd, 1.0, 1.0, seed, 5)[1] for seed in range(n)]
    torch.cuda.synchronize()
    cnt = np.bincount(torch.stack([o[0] for o in outs]).cpu().numpy(), minlength=6)
    chi2 = ((cnt - n * p) ** 2 / (n * p)).sum()
    assert chi2 < 25.7


def _chain_with_branches(T, V, r):
    """A path through every second node: deeper than what is taken ahead of the walk, one dead end per level."""
    par = np.array([-1] + [max(0, (i - 1) // 2 * 2) for i in range(1, T)], np.int32)
    return r.integers(0, V, T).astype(np.int32), par


@pytest.mark.parametrize("V,T,tree", [(4097, 4, "best"), (4097, 4096, "best"), (5001, 300, "chain"), (20000, 64, "best"),
                                      (32768, 65, "uniform"), (32769, 65, "best"), (50002, 700, "best"), (131072, 90, "chain")])
@pytest.mark.parametrize("ratio", [False, True])
@pytest.mark.parametrize("t,top_p,floor", [(0.6, 0.9, -12.0), (1.0, 1.0, -12.0), (1.0, 0.9, 0.0), (0.0, 1.0, -12.0)])
def test_walk_by_many_workgroups_is_the_walk_by_one(sx, V, T, tree, ratio, t, top_p, floor):
    """A workspace without room for the records and scratch rows takes the walk by one workgroup; with room, steps are taken
    at many nodes at once.  Same step, so the same bits: paths within the first 64 nodes and past them, rows that need the
    scratch row, rows too flat to be taken ahead (floor 0), paths deeper than what is taken ahead, and child tokens outside
    the vocabulary, which count only where the walk comes by."""
    r = np.random.default_rng(V + T)
    if tree == "chain":
        tok, par = _chain_with_branches(T, V, r)
    elif tree == "uniform":
        tok, par = wl.gen_uniform_tree(T, V, seed=V)
    else:
        tok, par, _ = wl.gen_best_first_tree(T, 8, V, seed=V + T, max_depth=24)
    tok, par = np.array(tok, np.int32), np.array(par, np.int32)
    g = torch.Generator(device=dev()).manual_seed(V)
    logits = torch.randn((T, V), generator=g, device=dev()) + floor
    depth = np.zeros(T, int)
    for i in range(1, T):
        depth[i] = depth[par[i]] + 1
    likely = {int(par[i]): i for i in range(1, T)}  # of every inner node one child, on the way to the deepest node where it can be
    i = int(depth.argmax())
    while par[i] >= 0:
        likely[int(par[i])] = i
        i = int(par[i])
    inner = np.array(sorted(likely))
    logits[to_dev(inner), to_dev(tok[[likely[i] for i in inner]].astype(np.int64))] = 9.0
    draft = torch.softmax(logits + 0.5 * torch.randn((T, V), generator=g, device=dev()), dim=1) if ratio else None
    td, pd = to_dev(tok), to_dev(par)
    many = sx.lib.sx_accept_walk_workspace(T, V)
    one = sx.lib.sx_accept_walk_workspace(1, V)
    assert many > one
    longest = 0
    for seed in range(6):
        got = []
        for size in (many, one):
            ws = torch.full((size,), 255, dtype=torch.uint8, device=dev())
            path, toks, n, _ = sx.accept_walk(logits, td, pd, t, top_p, seed, 11, draft_probs=draft, workspace=ws)
            n = int(n.item())
            got.append((path[:n].tolist(), toks[:n].tolist(), sx.lib.sx_check_status(ws.data_ptr(), None)))
        assert got[0] == got[1], (seed, got)
        assert got[0][2] == 0
        longest = max(longest, len(got[0][0]))
    if floor < 0 and t < 1 and not ratio:
        assert longest == depth.max() + 1
    if ratio:  # a bad token below a node that the walk visits is reported, elsewhere it is not
        path = got[0][0]
        kids = [i for i in range(1, T) if par[i] == path[0]]
        away = [i for i in range(1, min(T, 64)) if par[i] not in path]
        for bad, want in [(kids[0], -6)] + ([(away[0], 0)] if away else []):
            t2 = tok.copy()
            t2[bad] = V
            for size in (many, one):
                ws = torch.full((size,), 255, dtype=torch.uint8, device=dev())
                sx.accept_walk(logits, to_dev(t2), pd, t, top_p, 5, 11, draft_probs=draft, workspace=ws)
                assert sx.lib.sx_check_status(ws.data_ptr(), None) == want


@pytest.mark.parametrize("V,T", [(5001, 64), (5001, 700), (40000, 100)])
def test_walk_believes_nothing_that_was_in_the_workspace(sx, V, T):
    """The workgroups of a walk meet in words of the workspace, which nobody clears: what an earlier walk over other logits has
    left there, or anything else -- here records of every node with a wrong token and end, under a board that has begun, walked
    to a node or ended, and under all tags that this walk may choose -- changes no result, call after call."""
    tok, par, _ = wl.gen_best_first_tree(T, 8, V, seed=V + T, max_depth=24)
    td, pd = to_dev(np.array(tok, np.int32)), to_dev(np.array(par, np.int32))
    many, one = sx.lib.sx_accept_walk_workspace(T, V), sx.lib.sx_accept_walk_workspace(1, V)
    g = torch.Generator(device=dev()).manual_seed(T)
    logits = []
    for likely in range(3):
        x = torch.randn((T, V), generator=g, device=dev()) - 12.0
        kids = {}
        for i in range(1, T):
            kids.setdefault(int(par[i]), []).append(i)
        for p, c in kids.items():
            x[p, int(tok[c[likely % len(c)]])] = 9.0
        logits.append(x)
    words = min(T, 128)
    node = np.concatenate([np.arange(min(T, 64)), np.arange(64, words)]).astype(np.uint64)
    ws = torch.zeros(many, dtype=torch.uint8, device=dev())
    ws1 = torch.zeros(one, dtype=torch.uint8, device=dev())
    for r in range(30):
        if r >= 6:
            tags = np.full(words, 7 * r) if r % 2 else 500 + np.arange(words)
            fake = tags.astype(np.uint64) << np.uint64(48) | node << np.uint64(33) | np.uint64(77 << 2)
            child = [0, 6, 4096, 8191][r // 4 % 4] << 20  # none, a node, the last one there can be, one past every tree
            board = [0, 1 | child, 2, 1 | child | 5 << 2][r % 4] | int(tags[0]) << 48
            fake[0] = board
            ws[one:one + 8 * words] = torch.from_numpy(fake.view(np.uint8)).to(dev())
        x = logits[r % 3]
        path, toks, n, _ = sx.accept_walk(x, td, pd, 0.6, 0.9, r, 3, workspace=ws)
        p1, t1, n1, _ = sx.accept_walk(x, td, pd, 0.6, 0.9, r, 3, workspace=ws1)
        n, n1 = int(n.item()), int(n1.item())
        assert n == n1 and path[:n].tolist() == p1[:n].tolist() and toks[:n].tolist() == t1[:n].tolist(), r


# ------------------------------------------------------------------------------------------------
# acceptance by the ratio of target and draft probability (Sect. 4.1, "Comparison to speculative
# decoding"): sx_accept_walk with draft_probs against oracle.specinfer_walk
# ------------------------------------------------------------------------------------------------

def _sampled_tree(T, V, n_children, seed):
    """A tree whose children were drawn from a draft distribution, with that distribution per node and target
    logits that agree with it only roughly: draft rows = softmax of N(0,1) noise with a few lifted tokens; every
    node (breadth first, until T nodes) draws n_children tokens independently from its row (equal draws stay
    separate children); target logits = draft logits + N(0, 1.5) noise."""
    r = np.random.default_rng(seed)
    tokens, parent, rows = [int(r.integers(V))], [-1], []
    i = 0
    while i < len(tokens):
        lg = r.standard_normal(V)
        lift = r.choice(V, size=min(5, V), replace=False)
        lg[lift] += np.log(V) + r.uniform(2.0, 6.0, size=len(lift))   # the lifted tokens hold most of the mass at any V
        q = np.exp(lg - lg.max())
        q /= q.sum()
        rows.append((lg, q))
        if len(tokens) < T:
            for x in r.choice(V, size=min(n_children, T - len(tokens)), p=q):
                tokens.append(int(x))
                parent.append(i)
        i += 1
    draft_probs = np.stack([q for _, q in rows]).astype(np.float32)
    target = np.stack([lg for lg, _ in rows]) + 1.5 * r.standard_normal((len(rows), V))
    return np.array(tokens, np.int32), np.array(parent, np.int32), target.astype(np.float32), draft_probs


SI_MARGIN = 1e-5   # probabilities are at most one and carry ~1e-6 of absolute fp32 error


def _si_safe(ref):
    return all(min(m["m_acc"], m["m_u"]) > SI_MARGIN for m in ref["margins"])


@pytest.mark.parametrize("V,T,kids", [(1000, 40, 3), (32000, 60, 4), (50000, 24, 2), (64, 30, 3)])
@pytest.mark.parametrize("t,top_p", [(0.6, 0.9), (1.0, 1.0), (0.0, 1.0)])
def test_ratio_acceptance_matches_oracle(sx, V, T, kids, t, top_p):
    tok, par, target, dq = _sampled_tree(T, V, kids, seed=V + T)
    ld, qd, td, pd = to_dev(target), to_dev(dq), to_dev(tok), to_dev(par)
    checked = accepted = 0
    for seed in range(24):
        ref = oracle.specinfer_walk(target, dq, tok, par, t, top_p, seed=seed, pos0=31)
        if not _si_safe(ref):
            continue
        path, toks, n, ws = sx.accept_walk(ld, td, pd, t, top_p, seed, 31, draft_probs=qd)
        torch.cuda.synchronize()
        n = int(n.item())
        assert sx.check_status(ws) == 0
        assert path[:n].cpu().tolist() == ref["path"], (seed, ref)
        assert toks[:n].cpu().tolist() == ref["tokens"]
        checked += 1
        accepted += len(ref["path"]) - 1
    assert checked >= 12 and accepted >= 4        # the walks do go down the tree: target and draft agree roughly


@pytest.mark.parametrize("V", [1000, 32000, 50000])
@pytest.mark.parametrize("c", [65, 300, 1000])
def test_ratio_acceptance_over_lists_of_any_length(sx, V, c):
    """Targets with c possible tokens (the others masked out), more than one wave holds and fewer than the list's end, and
    children that are mostly rejected: the distribution goes through several rejections before it is drawn from."""
    T = 24
    tok, par, target, dq = _sampled_tree(T, V, 6, seed=V + c)
    r = np.random.default_rng(c)
    for i in range(T):
        keep = np.concatenate([np.argsort(-dq[i])[:6], r.choice(V, size=c, replace=False)])[:c]
        row = np.full(V, -np.inf, np.float32)
        row[keep] = r.normal(0.0, 2.0, size=len(keep))
        target[i] = row
    ld, qd, td, pd = to_dev(target), to_dev(dq), to_dev(tok), to_dev(par)
    checked = 0
    for seed in range(16):
        ref = oracle.specinfer_walk(target, dq, tok, par, 0.7, 1.0, seed=seed, pos0=31)
        if not _si_safe(ref):
            continue
        path, toks, n, _ = sx.accept_walk(ld, td, pd, 0.7, 1.0, seed, 31, draft_probs=qd)
        torch.cuda.synchronize()
        n = int(n.item())
        assert path[:n].cpu().tolist() == ref["path"] and toks[:n].cpu().tolist() == ref["tokens"], (seed, ref)
        checked += 1
    assert checked >= 8


def test_ratio_acceptance_emits_the_target_distribution(sx):
    """chi-square on the device: k children drawn from q by numpy; the first emitted token must follow p."""
    p = np.array([0.02, 0.4, 0.08, 0.25, 0.05, 0.2])
    q = np.array([0.3, 0.1, 0.25, 0.05, 0.2, 0.1])
    k, n = 3, 4000
    r = np.random.default_rng(5)
    ld = to_dev(np.tile(np.log(p).astype(np.float32), (k + 1, 1)))
    qd = to_dev(np.tile(q.astype(np.float32), (k + 1, 1)))
    pd = to_dev(np.array([-1] + [0] * k, np.int32))
    outs = []
    for seed in range(n):
        td = to_dev(np.array([0] + list(r.choice(6, size=k, p=q)), np.int32))
        outs.append(sx.accept_walk(ld, td, pd, 1.0, 1.0, seed, 5, draft_probs=qd)[1])
    torch.cuda.synchronize()
    cnt = np.bincount(torch.stack([o[0] for o in outs]).cpu().numpy(), minlength=6)
    chi2 = ((cnt - n * p) ** 2 / (n * p)).sum()
    assert chi2 < 25.7, (chi2, cnt / n)


def test_ratio_acceptance_special_cases(sx):
    p = np.array([0.02, 0.4, 0.08, 0.25, 0.05, 0.2])
    # draft == target: every first child is accepted, down the chain; then one token past the leaf
    tok, par = np.array([3, 1, 4, 1], np.int32), np.array([-1, 0, 1, 2], np.int32)
    rows = np.tile(np.log(p).astype(np.float32), (4, 1))
    for seed in range(8):
        path, toks, n, _ = sx.accept_walk(to_dev(rows), to_dev(tok), to_dev(par), 1.0, 1.0, seed, 2,
                                          draft_probs=to_dev(np.tile(p.astype(np.float32), (4, 1))))
        torch.cuda.synchronize()
        assert int(n.item()) == 4 and path[:4].cpu().tolist() == [0, 1, 2, 3] and toks[:3].cpu().tolist() == [1, 4, 1]
    # a child token outside the vocabulary is reported, not indexed
    bad = np.array([3, 99], np.int32)
    _, _, _, ws = sx.accept_walk(to_dev(rows[:2]), to_dev(bad), to_dev(np.array([-1, 0], np.int32)), 1.0, 1.0, 0, 0,
                                 draft_probs=to_dev(np.tile(p.astype(np.float32), (2, 1))))
    assert sx.check_status(ws) == -6
