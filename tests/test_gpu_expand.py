"""GPU parity: sx_expand_topk / sx_row_logsoftmax_topk against the oracle (Alg. 2, selectBest)."""
import numpy as np
import pytest
import torch

import oracle
import workloads as wl
from helpers import dev, to_dev

pytestmark = pytest.mark.gpu

LOGP_TOL = 2e-5      # fp32 log-sum-exp over <= 131072 terms vs fp64: a few 1e-6 in practice
SCORE_EPS = 1e-4     # two candidates closer than this may swap places (fp32-path tolerance)


@pytest.fixture(scope="module")
def sx():
    import paper_2406_02532_amd as m
    return m


def _run(sx, logits, cum, k, B):
    r, t, s, n, _ = sx.expand_topk(to_dev(logits), to_dev(cum), k, B)
    torch.cuda.synchronize()
    n = int(n.item())
    return r[:n].cpu().numpy(), t[:n].cpu().numpy(), s[:n].cpu().numpy(), n


def _check_rows(sx, logits, k):
    lp, idx = sx.row_logsoftmax_topk(to_dev(logits), k)
    torch.cuda.synchronize()
    ref_idx = oracle.row_topk(logits, k)
    ref_lp = np.take_along_axis(oracle.log_softmax(logits), ref_idx, -1)
    np.testing.assert_array_equal(idx.cpu().numpy(), ref_idx)             # bit-exact: raw-logit order, ties by id
    got = lp.cpu().numpy().astype(np.float64)
    finite = np.isfinite(ref_lp)
    assert np.array_equal(np.isneginf(got), np.isneginf(ref_lp))
    assert np.abs(got[finite] - ref_lp[finite]).max() <= LOGP_TOL


def _check_global(got, ref, B, n_cand):
    """Order and membership are unique except among candidates whose fp32 scores differ by less
    than SCORE_EPS from a neighbour / from the cut: compare exactly where the oracle's margins allow,
    otherwise compare the unique part and check that the rest is valid."""
    r, t, s, n = got
    assert n == min(B, n_cand) == len(ref["row"])
    np.testing.assert_allclose(s, ref["score"], atol=SCORE_EPS)
    assert np.all(np.diff(s) <= 0)
    ref_pairs = list(zip(ref["row"].tolist(), ref["token"].tolist()))
    got_pairs = list(zip(r.tolist(), t.tolist()))
    if got_pairs == ref_pairs:
        return
    # pairs may differ only inside runs of near-equal scores or across a near-tied cut
    sure = ref["score"] > ref["threshold"] + SCORE_EPS
    assert set(p for p, ok in zip(ref_pairs, sure) if ok) <= set(got_pairs)
    gaps = np.abs(np.diff(ref["score"]))
    for i, (a, b) in enumerate(zip(got_pairs, ref_pairs)):
        if a != b:
            near = (i > 0 and gaps[i - 1] < SCORE_EPS) or (i < len(gaps) and gaps[i] < SCORE_EPS) or not sure[i]
            assert near, f"position {i}: {a} vs {b} with no near-tie to excuse it"


def test_tiny_config_bit_exact(sx):
    """N=64 rows, V=1024, k=4, B=16 (the tiny configuration): exact result, margins checked."""
    for seed in range(5):
        logits, cum = wl.gen_expand_inputs(64, 1024, seed=seed, max_depth=8)
        ref = oracle.expand_topk(logits, cum, 4, 16)
        if ref["m_B"] < SCORE_EPS or ref["m_k"] <= 0:
            continue
        r, t, s, n = _run(sx, logits, cum, 4, 16)
        assert n == 16
        np.testing.assert_array_equal(r, ref["row"])
        np.testing.assert_array_equal(t, ref["token"])
        np.testing.assert_allclose(s, ref["score"], atol=LOGP_TOL)
        return
    pytest.fail("no seed with a safe margin")


@pytest.mark.parametrize("V,k", [(10, 3), (10, 10), (1001, 7), (1024, 64), (4096, 1), (5000, 100), (16384, 32),
                                 (32000, 32), (32000, 256), (50257, 8), (65536, 32), (128256, 32), (131072, 64)])
def test_row_topk_shapes(sx, V, k):
    N = 9
    logits, _ = wl.gen_expand_inputs(N, V, seed=V + k)
    _check_rows(sx, logits, k)


# Vocabularies too large for registers: a row to a workgroup of 1024 lanes up to a row per compute unit and 64 wanted, of
# 512 otherwise.  Odd widths (no 16-byte rows), one entry past a pass of all lanes, both sides of each line.
@pytest.mark.parametrize("N,V,k", [(1, 32769, 5), (2, 65540, 256), (3, 49153, 64), (3, 49153, 65), (256, 33000, 65), (256, 33000, 64),
                                   (257, 33001, 32), (300, 33000, 100)])
def test_row_topk_streamed_rows(sx, N, V, k):
    logits, _ = wl.gen_expand_inputs(N, V, seed=V + k)
    logits[0, 100:160] = logits[0].max()              # ties at the top
    _check_rows(sx, logits, k)


def test_row_topk_ties_and_degenerate_rows(sx):
    V = 32000
    logits, _ = wl.gen_expand_inputs(6, V, seed=77)
    logits[0, :] = 0.0                               # everything ties: the k lowest ids win
    logits[1, :] = np.round(logits[1, :])            # heavy ties on a coarse grid
    logits[2, 1000:1040] = logits[2].max() + 1.0     # 40 tied maxima, k = 32 cuts through them
    logits[3, ::2] = -np.inf                         # half the row masked out
    logits[4, :] = -np.arange(V, dtype=np.float32)   # sorted: one lane holds every winner
    logits[5, :] = np.where(np.arange(V) % 2 == 0, 0.0, -0.0)   # signed zeros compare equal
    _check_rows(sx, logits, 32)
    small = np.zeros((3, 40), dtype=np.float32)
    _check_rows(sx, small, 40)


def test_global_select_edge_cases(sx):
    logits, cum = wl.gen_expand_inputs(5, 300, seed=5)
    ref = oracle.expand_topk(logits, cum, 6, 1000)                 # B > N*k: everything, sorted
    _check_global(_run(sx, logits, cum, 6, 1000), ref, 1000, 30)
    ref = oracle.expand_topk(logits, cum, 6, 1)
    _check_global(_run(sx, logits, cum, 6, 1), ref, 1, 30)
    z = np.zeros((4, 64), dtype=np.float32)                        # all candidates tie: lowest flat index first
    r, t, s, n = _run(sx, z, np.zeros(4, np.float32), 8, 10)
    ref = oracle.expand_topk(z, np.zeros(4, np.float32), 8, 10)
    np.testing.assert_array_equal(r, ref["row"])
    np.testing.assert_array_equal(t, ref["token"])
    one = wl.gen_expand_inputs(1, 2000, seed=6)                    # a single row
    ref = oracle.expand_topk(one[0], one[1], 16, 8)
    _check_global(_run(sx, one[0], one[1], 16, 8), ref, 8, 16)


@pytest.mark.parametrize("N,k,B", [(1, 1, 1), (100, 32, 2048), (128, 32, 4096), (129, 32, 1), (500, 32, 8192), (512, 32, 700), (513, 32, 2048), (2048, 32, 2000),
                                   (513, 32, 8191), (33, 255, 1025), (2048, 32, 2048), (2047, 32, 2047), (2049, 32, 64),
                                   (600, 100, 4096)])
@pytest.mark.parametrize("spread", ["wide", "narrow", "rounded", "dead", "equal", "late"])
def test_global_select_sizes_and_spreads(sx, N, k, B, spread):
    """Candidate counts around what the select kernel holds per lane (4096 and 16384) and as codes (65536), every size of
    winner list, and scores over one octave, over many, with long ties, with dead rows (-inf) among the winners, all
    equal, and with ties that start behind the first 4096 candidates."""
    logits, cum = wl.gen_expand_inputs(N, 400, seed=N + k)
    if spread == "narrow":
        cum = (-1000.0 + cum * 1e-3).astype(np.float32)
    elif spread == "rounded":
        logits, cum = np.round(logits), np.round(cum).astype(np.float32)
    elif spread == "dead":
        cum[N // 3:] = -np.inf
    elif spread == "equal":
        logits, cum = np.zeros_like(logits), np.zeros_like(cum)
    elif spread == "late":
        logits, cum = np.zeros_like(logits), np.full_like(cum, -3.0)
        cum[:N // 2] = -4.0 - np.arange(N // 2, dtype=np.float32) / N
        cum[0] = -2.0
    ld, cd = to_dev(logits), to_dev(cum)
    lp, idx = sx.row_logsoftmax_topk(ld, k)
    r, t, s, n = _run(sx, logits, cum, k, B)
    m = min(B, N * k)
    score = (torch.from_numpy(cum)[:, None] + lp.cpu()).numpy().reshape(-1)      # the fp32 values the kernel orders
    order = np.lexsort((np.arange(N * k), -score))[:m]
    assert int(n) == m
    np.testing.assert_array_equal(r[:m], order // k)
    np.testing.assert_array_equal(t[:m], idx.cpu().numpy().reshape(-1)[order])
    np.testing.assert_array_equal(s[:m], score[order])


def test_many_rows_memory_path(sx):
    """N*k above 512*128: the select kernel walks candidates from memory instead of registers."""
    logits, cum = wl.gen_expand_inputs(3000, 256, seed=9)
    ref = oracle.expand_topk(logits, cum, 32, 4096)
    _check_global(_run(sx, logits, cum, 32, 4096), ref, 4096, 96000)


def test_full_size_draft_expansion(sx):
    """2048 rows x 32000 logits, k=32, then the best 2048 of 65536 candidates -- the launch
    configuration the benchmark times."""
    c = wl.CONFIGS["C4"]
    logits, cum = wl.gen_expand_inputs(c["N"], c["V"], seed=1234, std=c["std"], max_depth=c["max_depth"])
    ref = oracle.expand_topk(logits, cum, c["k"], c["B"])
    dl = to_dev(logits)
    lp, idx = sx.row_logsoftmax_topk(dl, c["k"])
    torch.cuda.synchronize()
    np.testing.assert_array_equal(idx.cpu().numpy(), ref["topk_idx"])
    assert np.abs(lp.cpu().numpy() - ref["topk_logp"]).max() <= LOGP_TOL
    got = _run(sx, logits, cum, c["k"], c["B"])
    _check_global(got, ref, c["B"], c["N"] * c["k"])
    # a child is never likelier than its parent (App. A)
    assert np.all(got[2] <= cum[got[0]] + 1e-6)
    # same inputs, same answer: the kernels have no order-dependent arithmetic
    again = _run(sx, logits, cum, c["k"], c["B"])
    for a, b in zip(got[:3], again[:3]):
        np.testing.assert_array_equal(a, b)


@pytest.mark.parametrize("N,V,k", [(600, 32000, 32), (513, 16388, 8), (700, 32768, 100), (1030, 20000, 64)])
def test_many_rows_of_a_large_vocabulary(sx, N, V, k):
    """More rows than the chip holds workgroups at a time (several rounds per compute unit) at vocabularies of
    16k-32k: ragged row counts, a vocabulary that is not a multiple of the lanes' share, k above the one-wave
    ordering, and rows that need the exact search in the middle of the launch; every row must come out as the
    oracle's."""
    logits, _ = wl.gen_expand_inputs(N, V, seed=N + V)
    logits[N - 1, :] = 1.5                            # the last row: all ties
    logits[N // 2, :] = np.round(logits[N // 2, :])   # heavy ties in the middle of the launch
    logits[300, ::3] = -np.inf
    logits[301, 7:7 + k + 5] = logits[301].max() + 2.0   # k cuts through a run of tied maxima
    _check_rows(sx, logits, k)


def test_shape_errors(sx):
    x = torch.zeros((4, 100), device=dev())
    c = torch.zeros(4, device=dev())
    with pytest.raises(sx.SxError) as e:
        sx.expand_topk(x, c, 101, 4)
    assert e.value.code == -2
    with pytest.raises(sx.SxError) as e:
        sx.expand_topk(x, c, 4, 9000)
    assert e.value.code == -2


@pytest.mark.parametrize("N,k", [(1, 1), (3, 5), (16, 16), (257, 1), (32, 32), (25, 41), (64, 64), (128, 64), (8193, 1)])
@pytest.mark.parametrize("ties", [False, True])
def test_selection_among_few_candidates(sx, N, k, ties):
    """Up to 256 candidates learn their places in one workgroup, up to 8192 in many, more as a sampled set: order by score, ties
    to the lower flat index, for as many picks as there are and for fewer."""
    V = 300
    r = np.random.default_rng(N * 100 + k)
    logits = r.standard_normal((N, V)).astype(np.float32)
    if ties:
        logits[:] = np.round(logits[:1])
        logits[N // 2:, 7:] = -np.inf
    cum = np.zeros(N, np.float32) if ties else -r.exponential(2.0, N).astype(np.float32)
    lp, idx = sx.row_logsoftmax_topk(to_dev(logits), k)
    flat = (lp.cpu().numpy() + cum[:, None]).reshape(-1)
    order = np.argsort(-flat, kind="stable")
    for B in {1, max(1, N * k // 2), min(N * k, 8192), min(N * k + 3, 8192)}:
        row, tok, score, n = _run(sx, logits, cum, k, B)
        assert n == min(B, N * k)
        want = order[:n]
        np.testing.assert_array_equal(row, want // k)
        np.testing.assert_array_equal(tok, idx.cpu().numpy().reshape(-1)[want])
        np.testing.assert_array_equal(score, flat[want])


@pytest.mark.parametrize("N,k", [(64, 4), (300, 4), (512, 16), (513, 16), (2048, 32), (5000, 128)])
@pytest.mark.parametrize("B", [3, 200])
def test_nan_scores_have_one_place_at_every_size(sx, N, k, B):
    """A score that is NaN is ordered by its bit pattern, before every number without the sign and behind -inf with it,
    whichever way the picks are selected (few candidates, all in the set, a sampled set, one workgroup), and the order of the
    others does not change."""
    V = 300
    r = np.random.default_rng(N + B)
    logits = r.standard_normal((N, V)).astype(np.float32)
    cum = -r.exponential(2.0, N).astype(np.float32)
    first, last = N // 3, N // 2
    cum[first] = np.nan
    cum[last:last + 2] = np.array([0xFFC00000], np.uint32).view(np.float32)[0]
    lp, idx = sx.row_logsoftmax_topk(to_dev(logits), k)
    flat = lp.cpu().numpy() + np.where(np.isnan(cum), 0.0, cum).astype(np.float32)[:, None]
    flat[first], flat[last:last + 2] = np.inf, -np.inf
    order = np.argsort(-flat.reshape(-1), kind="stable")
    row, tok, score, n = _run(sx, logits, cum, k, B)
    want = order[:min(B, N * k)]
    assert n == len(want)
    np.testing.assert_array_equal(row, want // k)
    np.testing.assert_array_equal(tok, idx.cpu().numpy().reshape(-1)[want])
    assert np.isnan(score[row == first]).all() and not np.isnan(score[(row != first) & (row != last) & (row != last + 1)]).any()


def test_share_of_a_selecting_workgroup_fits_its_list():
    """Flat indices are dealt to the selecting workgroups by a hash; whatever the scores, none gets more than its list holds."""
    bits = (np.arange(1 << 19, dtype=np.uint64) * 2654435761 & 0xFFFFFFFF) >> 16
    for blocks, upto in ((64, 2048), (128, 4096), (256, 8192), (128, 1 << 18), (256, 1 << 19)):
        assert np.bincount((bits[:upto] & (blocks - 1)).astype(np.int64)).max() <= min(4096, upto // blocks + 16)


@pytest.mark.parametrize("n,B", [(8193, 2048), (262144, 6144), (262145, 1), (524288, 6144), (524289, 2048)])
@pytest.mark.parametrize("misled", [False, True])
def test_selection_by_samples_up_to_its_limit(sx, n, B, misled):
    """Sampled sets of one candidate per row, to the last size that takes one and past it.  misled: the samples are all low and
    hide that nearly every candidate is above the threshold they set; the set is given up, and the picks are the same."""
    r = np.random.default_rng(n + B)
    cum = r.standard_normal(n).astype(np.float32)
    if misled:
        i = np.arange(4096, dtype=np.uint64)
        lo, hi = i * n // 4096, (i + 1) * n // 4096
        cum[lo + (i * 2654435761 % (1 << 32) >> 8) % (hi - lo)] -= 60.0
    logits = np.zeros((n, 2), np.float32)
    row, tok, score, got = _run(sx, logits, cum, 1, B)
    flat = sx.row_logsoftmax_topk(to_dev(logits[:1]), 1)[0].cpu().numpy()[0, 0] + cum
    want = np.argsort(-flat, kind="stable")[:B]
    assert got == B and not tok.any()
    np.testing.assert_array_equal(row, want)
    np.testing.assert_array_equal(score, flat[want])


@pytest.mark.parametrize("n,B", [(4097, 40), (8193, 8192), (16384, 6144), (16385, 40), (24577, 6144), (131073, 2000)])
@pytest.mark.parametrize("kind", ["equal", "few above", "dead", "dead and signed nan", "two values", "close"])
def test_ties_at_the_threshold_fill_the_picks_in_index_order(sx, n, B, kind):
    """More candidates of one score, -inf among them, than there are places: those above it first, then the lowest indices,
    wherever they lie and whichever form selects."""
    r = np.random.default_rng(n + B)
    cum = np.full(n, -3.5, np.float32)
    if kind == "few above":
        at = r.choice(n, B // 3, replace=False)
        cum[at] = -3.5 + r.integers(1, 50, B // 3).astype(np.float32) / 16
    elif kind.startswith("dead"):
        cum[:] = -np.inf
        live = r.choice(n, B // 2, replace=False)
        cum[live] = r.standard_normal(B // 2).astype(np.float32)
        if kind != "dead":  # so many that the -inf do not fill the picks
            rest = np.setdiff1d(np.arange(n), live)
            cum[rest[:len(rest) - B // 4]] = np.array([0xFFC00000], np.uint32).view(np.float32)[0]
    elif kind == "two values":
        cum[r.random(n) < 0.5] = 0.0
        cum[r.random(n) < 0.1] = -0.0
    elif kind == "close":
        cum += 1e-6 * r.integers(0, 4, n).astype(np.float32)
    logits = np.zeros((n, 2), np.float32)
    row, tok, score, got = _run(sx, logits, cum, 1, B)
    flat = sx.row_logsoftmax_topk(to_dev(logits[:1]), 1)[0].cpu().numpy()[0, 0] + cum
    signed = np.isnan(flat)  # behind -inf
    want = np.argsort(np.where(signed, np.inf, -flat) + 0.0, kind="stable")
    if signed.any():
        want = np.concatenate([want[~signed[want]], np.flatnonzero(signed)])
    want = want[:B]
    assert got == B and not tok.any()
    np.testing.assert_array_equal(row, want)
    np.testing.assert_array_equal(score, flat[want])


@pytest.mark.parametrize("N,V,k", [(3, 32769, 1), (129, 32772, 32), (9, 40001, 56), (17, 65537, 32), (129, 65540, 4),
                                   (130, 131072, 32), (16, 100003, 32), (3, 131069, 33)])
def test_long_rows_shared_among_workgroups(sx, N, V, k):
    """Rows of more than 32768 entries, put together from their shares (2, 4 and 8 of them, V a multiple of 4 and not), have the
    tokens of the oracle in its order: equal entries across all shares, shares of -inf alone, the best at the edges of shares.
    A workspace without room for the shares takes the streaming kernel, with the same tokens."""
    rng = np.random.default_rng(V)
    logits = (rng.standard_normal((N, V)) * 3).astype(np.float32)
    logits[0] = 1.25
    logits[1] = -np.inf
    logits[1, [7, V // 2, V - 1]] = [0.5, 2.0, 0.5]
    for parts in (2, 4, 8):
        edge = ((V + parts - 1) // parts + 3) & ~3
        logits[2, [edge - 1, edge]] = 15.0 + 1.0 / parts
    # rows far enough apart that the selection of all candidates leaves each row's in their order
    spacing = 64.0
    cum = (-spacing * np.arange(N)).astype(np.float32)
    ref_idx = oracle.row_topk(logits, k)
    ref_lp = np.take_along_axis(oracle.log_softmax(logits), ref_idx, -1)
    shares = sx.lib.sx_expand_topk_workspace(N, V, k, N * k)
    least = 256 + 3 * ((N * k * 4 + 255) // 256 * 256)
    assert shares > least
    for nbytes in (shares, least):
        ws = torch.empty(nbytes, dtype=torch.uint8, device=dev())
        r, t, s, n, _ = sx.expand_topk(to_dev(logits), to_dev(cum), k, N * k, workspace=ws)
        r, t, s = r.cpu().numpy(), t.cpu().numpy(), s.cpu().numpy().astype(np.float64)
        assert int(n.item()) == N * k
        for i in range(N):
            at = r == i
            np.testing.assert_array_equal(t[at], ref_idx[i], err_msg=f"row {i}")
            got, want = s[at], ref_lp[i] + cum[i]
            fin = np.isfinite(want)
            assert np.array_equal(np.isneginf(got), ~fin)
            # the sum of score and log-probability rounds once at the size of the row's offset
            assert np.abs(got[fin] - want[fin]).max() <= LOGP_TOL + spacing * (N + 1) * 2.0 ** -24


@pytest.mark.parametrize("N,V,k", [(130, 131072, 32), (9, 40001, 56), (129, 32772, 1), (5, 100000, 100), (6, 32000, 32)])
def test_masked_rows(sx, N, V, k):
    """Rows of one low value (-inf, the lowest number, -1e9) but for a range of tokens: fewer than k, k, a few hundred, more than
    the candidates' slots, at the beginning, in the middle and at the end; shared among workgroups, streamed, and in registers."""
    rng = np.random.default_rng(V + k)
    logits = (rng.standard_normal((N, V)) * 3).astype(np.float32)
    lows = (-np.inf, np.finfo(np.float32).min, -1e9)
    for i, count in enumerate((1, k, 300, 1500, 2 * V // 3)):
        first = (0, V // 2, V - count, V // 4 - count // 2, 0)[i]
        kept = logits[i, first:first + count].copy()
        logits[i] = lows[i % 3]
        logits[i, first:first + count] = kept
    idx = oracle.row_topk(logits, k)
    lp = np.take_along_axis(oracle.log_softmax(logits), idx, -1)
    got_lp, got_idx = sx.row_logsoftmax_topk(to_dev(logits), k)
    np.testing.assert_array_equal(got_idx.cpu().numpy(), idx)
    rows = np.arange(N, dtype=np.float32)
    for nbytes in (sx.lib.sx_expand_topk_workspace(N, V, k, N * k), 256 + 3 * ((N * k * 4 + 255) // 256 * 256)):
        ws = torch.empty(nbytes, dtype=torch.uint8, device=dev())
        r, t, s, n, _ = sx.expand_topk(to_dev(logits), to_dev(-64.0 * rows), k, N * k, workspace=ws)
        r, t, s = r.cpu().numpy(), t.cpu().numpy(), s.cpu().numpy().astype(np.float64)
        assert int(n.item()) == N * k
        for i in range(N):
            np.testing.assert_array_equal(t[r == i], idx[i], err_msg=f"row {i}")
            want = lp[i] - 64.0 * i
            fin = np.isfinite(want)
            assert np.array_equal(np.isneginf(s[r == i]), ~fin)
            # the sum of score and log-probability rounds once, at its own size
            assert (np.abs(s[r == i][fin] - want[fin]) <= LOGP_TOL + np.abs(want[fin]) * 2.0 ** -22).all()


def test_masked_rows_take_no_longer(sx):
    """A third of every row masked, so that a whole share of it is: no more than three times the time of rows without a mask
    (fifty times, when such a share was searched bit by bit)."""
    N, V, k, B = 600, 128256, 32, 2048
    x = wl.hash_normal(5, (N, V), std=3.0, device=dev())
    masked = x.clone()
    masked[:, 2 * V // 3:] = -float("inf")
    cum = torch.zeros(N, device=dev())
    ws = torch.empty(sx.lib.sx_expand_topk_workspace(N, V, k, B), dtype=torch.uint8, device=dev())

    def us(t):
        best = 1e9
        for _ in range(5):
            e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            e[0].record()
            sx.expand_topk(t, cum, k, B, workspace=ws)
            e[1].record()
            e[1].synchronize()
            best = min(best, e[0].elapsed_time(e[1]))
        return best

    plain, with_mask = us(x), us(masked)
    assert with_mask <= 3 * plain, (plain, with_mask)


@pytest.mark.parametrize("N,V,k", [(256, 50000, 8), (200, 128256, 32), (64, 100003, 56)])
def test_log_sum_exp_of_shared_rows_is_rounded_once(sx, N, V, k):
    """Logits around 5000: value and log-sum-exp are multiples of 2^-12 and their difference is exact, so a score's error is the
    log-sum-exp's rounding, half a unit in its last place (2^-12), and a little for the sum before it."""
    logits = wl.hash_normal(77, (N, V), std=3.0, mean=5000.0, device=dev())
    r, t, s, n, _ = sx.expand_topk(logits, torch.zeros(N, device=dev()), k, N * k)
    want = torch.log_softmax(logits.double(), 1)[r.long(), t.long()]
    assert int(n.item()) == N * k
    assert float((s.double() - want).abs().max()) <= 2.0 ** -12 * 1.02
