"""The narrow GEMMs (at most 128 rows): every number of row blocks, every tile width, whole and with K cut."""
import numpy as np
import pytest
import torch

import workloads as wl
from helpers import bf16_ulp
from test_gpu_w4_model import test_paired_columns_of_4bit_products as check_pairs
from test_gpu_verify import dev, sx, test_qkv_projection_with_rotary_epilogue as check_qkv  # noqa: F401

# (mode, N, K, columns of a tile, K is cut) at 128 rows, with the workspace; ragged columns, K of one slab, of less than the
# stages hold, of one slab more than they hold twice over
SHAPES = [
    (0, 72, 64, 64, False), (0, 250, 1088, 64, True), (1, 1000, 2048, 64, True), (0, 16500, 192, 128, False),
    (1, 9000, 4096, 128, True), (2, 40, 64, 64, False), (2, 1500, 4096, 64, True), (2, 8200, 192, 96, False),
    (2, 5000, 4096, 96, True), (2, 14000, 320, 128, False),
]


def test_shapes_take_every_form(sx):
    ws = sx.lib.sx_gemm_bf16_workspace()
    for mode, N, K, columns, cut in SHAPES:
        got, parts = sx.gemm_bf16_narrow_plan(N, K, mode, ws)
        assert (got, parts > 1) == (columns, cut), (mode, N, K)


@pytest.mark.gpu
@pytest.mark.parametrize("M", [1, 16, 17, 32, 33, 64, 65, 80, 81, 112, 113, 128])
def test_row_blocks(sx, M):
    """At the edges of every number of row blocks, against the fp64 product: fp32 sums of K terms, rounded to bf16 once in the
    SwiGLU form.  Rows behind the last one stay untouched, and the workspace's counters are back at zero."""
    ws = torch.zeros(sx.lib.sx_gemm_bf16_workspace(), dtype=torch.uint8, device=dev())
    for mode, N, K, _, _ in SHAPES:
        X = wl.hash_normal(61, (M, K), dtype=torch.bfloat16, device=dev())
        W = wl.hash_normal(62, (N, K), std=0.05, dtype=torch.bfloat16, device=dev())
        g = X.double() @ W.double().T
        for work in (None, ws):
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


@pytest.mark.gpu
@pytest.mark.parametrize("T", [1, 16, 17, 40, 80, 100, 128])
def test_qkv_row_blocks(sx, T):
    """The rotating form: 64 columns, whole and cut; 96 (18432 columns whole, 12288 cut); 128."""
    for d, Hq, Hkv in ((64, 1, 1), (1088, 4, 2), (192, 112, 16), (4096, 32, 32), (2048, 64, 8)):
        check_qkv(sx, T, d, Hq, Hkv, None, None, None)


@pytest.mark.gpu
@pytest.mark.parametrize("M", [1, 16, 17, 32, 33, 64, 65, 80, 81, 112, 113, 128])
def test_row_blocks_4bit(sx, M):
    """The form with 4-bit weights at the same edges: 64 columns whole and cut, 96 whole and cut, 128 whole and cut, against the
    product with bf16(scale * (code - zero)) in 64 bits."""
    ws = torch.zeros(sx.lib.sx_gemm_w4a16_workspace(), dtype=torch.uint8, device=dev())
    for mode, N, K, group in ((0, 250, 384, 128), (1, 3072, 4096, 512), (0, 20500, 512, 64), (1, 12300, 4096, 128),
                              (0, 30010, 256, 256), (1, 10200, 8192, 128)):
        X = wl.hash_normal(64, (M, K), dtype=torch.bfloat16, device=dev())
        q, s, z = (t.to(dev()) for t in wl.gen_w4(N, K, group, seed=65))
        codes = torch.stack([(q >> (4 * j)) & 15 for j in range(8)], 2).reshape(N, K).float()
        W = (s.float().repeat_interleave(group, 1) * (codes - z.float().repeat_interleave(group, 1))).to(torch.bfloat16)
        want = X.double() @ W.double().T
        tol = 1e-5 * np.sqrt(K) * float(want.abs().max()) + 1e-6
        for work in (None, ws):
            Y = torch.full((M + 16, N), 7.0, dtype=torch.float32, device=dev())
            sx.gemm_w4a16_bf16(X, q, s, z, Y[:M], group, mode=mode, workspace=work)
            assert float((Y[:M].double() - want - (7.0 if mode == 1 else 0.0)).abs().max()) <= tol, (mode, N, K)
            assert bool((Y[M:] == 7.0).all())


@pytest.mark.gpu
@pytest.mark.parametrize("T", [16, 100])
def test_paired_4bit_columns_in_tiles_of_96(sx, T):
    check_pairs(sx, T, (1, 256, 128, 16, 128, 10240, 500))
