"""NaN in data: what reads it is NaN, at every form of a launch and whatever the memory held before; nothing else changes."""
import numpy as np
import pytest
import torch

import oracle
import workloads as wl
from helpers import dev, to_dev, weights_to

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sx():
    import paper_2406_02532_amd as m
    return m


@pytest.mark.parametrize("T,P", [(1, 70), (40, 300), (300, 65), (2048, 130)])
def test_attention_over_a_key_of_nan(sx, T, P):
    """One KV head's prefix key is NaN: its query heads' rows are NaN, the other heads' as without it; a NaN key of a node
    reaches its descendants alone, a NaN query its own row.  128-row and 64-row workgroups."""
    Hq, Hkv = 4, 2
    r = lambda key, n, h: wl.hash_normal(key, (n, h, 128), dtype=torch.bfloat16, device=dev())  # noqa: E731
    q, kt, vt, kp, vp = r(1, T, Hq), r(2, T, Hkv), r(3, T, Hkv), r(4, P, Hkv), r(5, P, Hkv)
    par = np.array([-1] + [(i - 1) // 2 for i in range(1, T)], np.int32)

    def run(q, kt, kp):
        out = torch.full_like(q, 7.0)
        return sx.tree_attention_bf16(q, kt, vt, kp, vp, to_dev(par), out=out)[0].cpu()

    clean = run(q, kt, kp)
    assert bool(torch.isfinite(clean.float()).all())
    bad = kp.clone()
    bad[P - 3, 1, 5] = float("nan")
    got = run(q, kt, bad)
    assert bool(torch.isnan(got[:, 2:].float()).all()) and torch.equal(got[:, :2], clean[:, :2])
    at = min(3, T - 1)
    bad = kt.clone()
    bad[at, 0, 0] = float("nan")
    got = run(q, bad, kp)
    below = np.zeros(T, bool)
    for i in range(T):
        below[i] = i == at or (par[i] >= 0 and below[par[i]])
    hit = torch.zeros(T, Hq, 128, dtype=torch.bool)
    hit[torch.from_numpy(below), :2] = True
    assert torch.equal(torch.isnan(got.float()), hit) and torch.equal(got[~hit], clean[~hit])
    bad = q.clone()
    bad[T - 1, 3, 127] = float("nan")
    got = run(bad, kt, kp)
    hit = torch.zeros(T, Hq, 128, dtype=torch.bool)
    hit[T - 1, 3] = True
    assert torch.equal(torch.isnan(got.float()), hit) and torch.equal(got[~hit], clean[~hit])


@pytest.mark.parametrize("P", [100, 1000])
def test_forward_of_a_small_batch_over_a_key_of_nan(sx, P):
    """The batch of a draft model, whose key tiles are shared among workgroups (1000 prefix keys) or not: every row is NaN,
    whether the workspace held zeros, small numbers or an earlier call's rows."""
    cfg = wl.ModelCfg(2, 512, 4, 2, 128, 1024, 1000, dtype="bf16")
    T = 100
    mw = sx.ModelWeights(cfg, weights_to(wl.gen_weights(cfg, seed=21), dev()))
    kv = lambda key: wl.hash_normal(key, (2, P, 2, 128), dtype=cfg.torch_dtype, device=dev())  # noqa: E731
    pk, pv = kv(31), kv(32)
    tok, par = wl.gen_uniform_tree(T, cfg.vocab, seed=3)
    clean, ws = sx.verify_tree(mw, pk, pv, to_dev(tok), to_dev(par))
    assert bool(torch.isfinite(clean).all())
    for layer in (0, 1):
        bad = pk.clone()
        bad[layer, 17, 0, 3] = float("nan")
        for fill in (None, 0, 0x3C):
            if fill is not None:
                ws.fill_(fill)
            got, _ = sx.verify_tree(mw, bad, pv, to_dev(tok), to_dev(par), workspace=ws)
            assert sx.check_status(ws) == 0
            assert bool(torch.isnan(got).all()), (layer, fill)


def _rows_with_nan(N, V, k):
    rng = np.random.default_rng(V + k)
    x = (rng.standard_normal((N, V)) * 3).astype(np.float32)
    x[0, V // 3] = np.nan
    x[1, :V // 8] = np.nan                       # a share of NaN alone
    x[2] = -np.inf
    x[2, 5], x[2, [0, V // 2, V - 1]] = np.nan, [1.0, 2.0, 1.0]
    x[3] = np.nan
    x[4] = np.nan
    x[4, [3, V - 2]] = [-1.0, 4.0]               # fewer numbers than picks
    x[5] = -np.inf
    x[5, V // 2:V // 2 + k - 1] = 1.5            # no NaN: the other picks are -inf
    x[6] = -np.inf
    x[6, V - 1] = np.nan
    x[7, V - V // 8:] = -np.inf
    x[7, V - 1] = np.nan                         # a NaN in a share of -inf
    nan = np.isnan(x).any(1)
    with np.errstate(invalid="ignore"):
        lp = np.take_along_axis(oracle.log_softmax(np.where(nan[:, None], 0, x)), oracle.row_topk(x, k), -1)
    lp[nan] = np.nan
    return x, oracle.row_topk(x, k), lp


@pytest.mark.parametrize("V,k", [(500, 7), (4096, 100), (9000, 64), (32768, 32), (40001, 8), (65540, 70), (131072, 200)])
def test_row_topk_of_rows_with_nan(sx, V, k):
    """NaN comes behind every number, by index, and the log-probabilities of a row that holds one are NaN: the register and the
    streaming kernel, small and large k.  Every place is written."""
    x, idx, lp = _rows_with_nan(9, V, k)
    got_lp = torch.full((9, k), 7.0, device=dev())
    got_idx = torch.full((9, k), -7, dtype=torch.int32, device=dev())
    sx.row_logsoftmax_topk(to_dev(x), k, topk_logp=got_lp, topk_idx=got_idx)
    np.testing.assert_array_equal(got_idx.cpu().numpy(), idx)
    np.testing.assert_allclose(got_lp.cpu().numpy(), lp, rtol=0, atol=1e-4)


@pytest.mark.parametrize("N,V,k", [(17, 65537, 32), (9, 40001, 56), (129, 65540, 8), (130, 131072, 32)])
def test_expansion_of_long_rows_with_nan(sx, N, V, k):
    """The same for rows shared among workgroups, and with a workspace that has no room for the shares."""
    x, idx, lp = _rows_with_nan(N, V, k)
    cum = np.zeros(N, np.float32)
    for nbytes in (sx.lib.sx_expand_topk_workspace(N, V, k, N * k), 256 + 3 * ((N * k * 4 + 255) // 256 * 256)):
        ws = torch.full((nbytes,), 0x3C, dtype=torch.uint8, device=dev())
        r, t, s, n, _ = sx.expand_topk(to_dev(x), to_dev(cum), k, N * k, workspace=ws)
        r, t, s = r.cpu().numpy(), t.cpu().numpy(), s.cpu().numpy()
        assert int(n.item()) == N * k
        for i in range(N):
            at = np.argsort(t[r == i])  # (rows with equal scores meet in the selection; a row's own order is tested above)
            np.testing.assert_array_equal(t[r == i][at], np.sort(idx[i]), err_msg=f"row {i}")
            np.testing.assert_allclose(s[r == i][at], lp[i][np.argsort(idx[i])], rtol=0, atol=1e-4, err_msg=f"row {i}")
