"""The narrow GEMMs (at most 128 rows): every number of row blocks, every tile width, whole and with K cut.  Which form a shape
takes at which number of rows, and that none is missing, is asserted on the CPU."""
import numpy as np
import pytest
import torch

import oracle
import workloads as wl
from gemm_shapes import NARROW_QKV_SHAPES, NARROW_SHAPES, ROW_BLOCK_EDGES, W4_PAIR_SHAPES, W4_SHAPES
from helpers import bf16_ulp, dev, to_dev
from test_gpu_w4_model import test_paired_columns_of_4bit_products as check_pairs
from test_gpu_verify import sx  # noqa: F401

pytestmark = pytest.mark.gpu

# shapes whose form changes with the rows: (mode, N, K), (K, query heads, KV heads), (N, K, group)
VARYING = [(0, 250, 1088), (1, 9000, 4096), (2, 5000, 4096)]
VARYING_QKV = [(1088, 4, 2), (4096, 32, 32), (2048, 64, 8)]
VARYING_W4 = [(12300, 4096, 128)]


@pytest.mark.parametrize("M", ROW_BLOCK_EDGES)
def test_row_blocks(sx, M):
    """At the edges of every number of row blocks, against the fp64 product: fp32 sums of K terms, rounded to bf16 once in the
    SwiGLU form; storing and adding to Y.  Rows behind the last one stay untouched, and the workspace's counters are back at
    zero."""
    ws = torch.zeros(sx.lib.sx_gemm_bf16_workspace(), dtype=torch.uint8, device=dev())
    for kind, N, K in [s[:3] for s in NARROW_SHAPES] + VARYING:
        X = wl.hash_normal(61, (M, K), dtype=torch.bfloat16, device=dev())
        W = wl.hash_normal(62, (N, K), std=0.05, dtype=torch.bfloat16, device=dev())
        g = X.double() @ W.double().T
        for mode, work in [(m, w) for m in ((2,) if kind == 2 else (0, 1)) for w in (None, ws)]:
            if mode == 2:
                W2 = wl.hash_normal(63, (N, K), std=0.05, dtype=torch.bfloat16, device=dev())
                Y = torch.full((M + 16, N), 7.0, dtype=torch.bfloat16, device=dev())
                sx.gemm_bf16(X, W, Y[:M], mode=2, W2=W2, workspace=work)
                want = (g / (1 + torch.exp(-g)) * (X.double() @ W2.double().T)).cpu().numpy()
                assert np.all(np.abs(Y[:M].double().cpu().numpy() - want) <= 0.51 * bf16_ulp(want) + 1e-5 * np.abs(want).max())
            else:
                Y = torch.full((M + 16, N), 7.0, dtype=torch.float32, device=dev())
                sx.gemm_bf16(X, W, Y[:M], mode=mode, workspace=work)
                tol = 1e-5 * np.sqrt(K) * float(g.abs().max()) + 1e-6
                assert float((Y[:M].double() - g - (7.0 if mode == 1 else 0.0)).abs().max()) <= tol, (mode, N, K)
            assert bool((Y[M:] == 7.0).all())
    assert int(ws[:1024].max()) == 0


@pytest.mark.parametrize("T", sorted({40, 100, *ROW_BLOCK_EDGES}))
def test_qkv_row_blocks(sx, T):
    """The rotating form, against the oracle's rope applied to fp64 projections, correctly rounded to bf16 up to fp32 sums."""
    pos = (np.arange(T) * 7 % 3000 + 5).astype(np.int32)
    for d, Hq, Hkv in [s[1:4] for s in NARROW_QKV_SHAPES] + VARYING_QKV:
        X = wl.hash_normal(11, (T, d), dtype=torch.bfloat16, device=dev())
        W = [wl.hash_normal(12 + i, (h * 128, d), std=0.05, dtype=torch.bfloat16, device=dev()) for i, h in enumerate((Hq, Hkv, Hkv))]
        got = sx.qkv_rope_bf16(X, *W, to_dev(pos), 10000.0)
        for i, (y, w) in enumerate(zip(got, W)):
            want = (X.double() @ w.double().T).cpu().numpy().reshape(T, -1, 128)
            if i < 2:
                want = oracle.rope(want, pos, 10000.0)
            err = np.abs(y.double().cpu().numpy() - want)
            assert np.all(err <= 0.51 * bf16_ulp(want) + 2e-5 * np.abs(want).max()), (d, Hq, Hkv, i)


def _w4(N, K, group, seed):
    """Codes, scales and zero points on the device, and bf16(scale * (code - zero))."""
    q, s, z = (t.to(dev()) for t in wl.gen_w4(N, K, group, seed=seed))
    codes = torch.stack([(q >> (4 * j)) & 15 for j in range(8)], 2).reshape(N, K).float()
    W = (s.float().repeat_interleave(group, 1) * (codes - z.float().repeat_interleave(group, 1))).to(torch.bfloat16)
    return q, s, z, W


@pytest.mark.parametrize("M", ROW_BLOCK_EDGES)
def test_row_blocks_4bit(sx, M):
    """The form with 4-bit weights at the same edges, against the product with bf16(scale * (code - zero)) in 64 bits, storing
    and adding to Y."""
    ws = torch.zeros(sx.lib.sx_gemm_w4a16_workspace(), dtype=torch.uint8, device=dev())
    for N, K, group in [s[:3] for s in W4_SHAPES] + VARYING_W4:
        X = wl.hash_normal(64, (M, K), dtype=torch.bfloat16, device=dev())
        q, s, z, W = _w4(N, K, group, 65)
        want = X.double() @ W.double().T
        tol = 1e-5 * np.sqrt(K) * float(want.abs().max()) + 1e-6
        for mode, work in ((0, None), (1, None), (0, ws), (1, ws)):
            Y = torch.full((M + 16, N), 7.0, dtype=torch.float32, device=dev())
            sx.gemm_w4a16_bf16(X, q, s, z, Y[:M], group, mode=mode, workspace=work)
            assert float((Y[:M].double() - want - (7.0 if mode == 1 else 0.0)).abs().max()) <= tol, (mode, N, K)
            assert bool((Y[M:] == 7.0).all())
    assert int(ws[:1024].max()) == 0


@pytest.mark.parametrize("T", [16, 100])
def test_paired_4bit_columns_in_tiles_of_96(sx, T):
    check_pairs(sx, T, (1, 256, 128, 16, 128, 10240, 500))


@pytest.mark.parametrize("d,Hq,Hkv,F", [s[:4] for s in W4_PAIR_SHAPES])
def test_row_blocks_of_paired_4bit_columns(sx, d, Hq, Hkv, F):
    """The QKV and SwiGLU forms with 4-bit weights, in a model of one layer, against the bf16 model with the dequantised weights,
    whose products are held to 64 bits above.  Both round q, k, v, the activations and the layer's inputs to bf16 at the same
    places, and in either a value may fall on the other side of a rounding: up to 5e-3 of a row (2-norms) measured over all of
    them, four times that allowed."""
    cfg, P, V = wl.ModelCfg(1, d, Hq, Hkv, 128, F, 500, dtype="bf16"), 20, 500
    shapes = dict(wq=(Hq * 128, d), wk=(Hkv * 128, d), wv=(Hkv * 128, d), wo=(d, Hq * 128), w_gate=(F, d), w_up=(F, d), w_down=(d, F))
    normal = lambda key, shape, std=1.0, mean=0.0: wl.hash_normal(key, shape, std=std, mean=mean, dtype=torch.bfloat16, device=dev())  # noqa: E731
    w4, bf = {}, {n: normal(71 + i, (d,), 0.1, 1.0) for i, n in enumerate(("attn_norm", "ffn_norm"))}
    norms = dict(bf)
    for i, (n, s) in enumerate(shapes.items()):
        *w4[n], bf[n] = _w4(*s, 128, 80 + i)
    ends = dict(embed=normal(73, (V, d)), final_norm=normal(74, (d,), 0.1, 1.0), lm_head=normal(75, (V, d), 0.02))
    m4 = sx.ModelWeights(cfg, dict(ends, layers=[norms], layers_w4=[w4], w4_group=128))
    m16 = sx.ModelWeights(cfg, dict(ends, layers=[bf]))
    pk, pv = normal(76, (1, P, Hkv, 128)), normal(77, (1, P, Hkv, 128))
    worst = 0.0
    for T in ROW_BLOCK_EDGES:
        tok, par = (to_dev(a) for a in wl.gen_uniform_tree(T, V, seed=3))
        kv = lambda: torch.zeros((1, T, Hkv, 128), dtype=torch.bfloat16, device=dev())  # noqa: E731
        outs = []
        for m in (m4, m16):
            k, v = kv(), kv()
            logits, ws = sx.verify_tree(m, pk, pv, tok, par, tree_k_out=k, tree_v_out=v)
            assert sx.check_status(ws) == 0
            outs.append((logits.double(), k.double(), v.double()))
        for a, b in zip(*outs):
            a, b = a.reshape(T, -1), b.reshape(T, -1)
            worst = max(worst, float(((a - b).norm(dim=1) / b.norm(dim=1)).max()))
    print(f"\n[paired 4-bit columns, d={d}] largest relative difference of a row {worst:.1e}")
    assert worst <= 2e-2
