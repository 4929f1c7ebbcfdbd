"""17 to 64 tokens of matrices tall enough for one column of the prompt kernel's tiles (tiles of 32 tokens for up to 32): both sides
of the rule's limits, ragged last tiles, rows of an odd number of groups and of fewer blocks than waves that share them."""
import copy

import numpy as np
import pytest
import torch

import oracle
import paper_2605_14844_amd as xfp
import xfp_inputs as xi
from helpers import gated_rel_err

pytestmark = pytest.mark.gpu
V2, V2A = xi.MODE_V2, xi.MODE_V2A


TILE = lambda M: (128, 32 if M <= 32 else 64)                         # of the prompt kernel; the 64-token kernel's has 32 rows


@pytest.mark.parametrize("mode,bits,N,K,M,tiles", [
    (V2, 4, 24577, 3200, 17, True), (V2, 4, 24576, 3200, 17, False), (V2A, 3, 24600, 1664, 32, True), (V2, 2, 24577, 128, 33, True), (V2A, 4, 24577, 384, 48, True),
    (V2, 3, 20481, 1152, 49, True), (V2, 3, 20480, 1152, 49, False), (V2A, 2, 20500, 256, 64, True), (V2, 3, 16385, 640, 33, True), (V2A, 2, 16400, 768, 61, True),
    (V2, 4, 16400, 1024, 64, True), (V2, 2, 57345, 1664, 25, True), (V2A, 3, 45057, 512, 40, True), (V2A, 3, 45057, 640, 40, False)])
def test_wide_calls_in_tiles(mode, bits, N, K, M, tiles):
    W = xi.random_weights(mode, bits, N, K, density=0.004, seed=N + K)
    x = xi.activations(np.random.default_rng(N + M), M, K)
    dW, xd = xfp.upload(W), torch.from_numpy(x.view(np.int16)).cuda().view(torch.float16)
    assert xfp.xfp_launch_route(dW, M) == (xfp.XFP_ROUTE_WIDE, M)
    assert xfp.xfp_wide_tile(dW, M) == (TILE(M) if tiles else (32, (M + 15) // 16 * 16))
    y = xfp.xfp_gemv(dW, xd, y_dtype=torch.float32)
    torch.cuda.synchronize()
    assert gated_rel_err(y.cpu().numpy().astype(np.float64), oracle.gemv_weights(W, x)) <= 1e-4      # fp32 results, as in the other kernels' tests
    for t in (torch.float16, torch.bfloat16):
        assert torch.equal(xfp.xfp_gemv(dW, xd, y_dtype=t), y.to(t))
    fixed = torch.full((M, N), 7.0, device="cuda")
    xfp.xfp_gemv_noalloc(dW, xd, fixed)
    assert torch.equal(fixed, y)


# rows of more than 64 groups, whose library ids are fetched in the loop, up to the longest that each tile takes (the other kernel's
# row beside it); no outliers, outliers in the last row alone
@pytest.mark.parametrize("mode,bits,N,K,M,density", [(V2A, 2, 24577, 8320, 20, 0.003), (V2A, 3, 24600, 16384, 32, 0.001), (V2A, 4, 24577, 12416, 17, 0.0), (V2, 4, 24577, 16384, 24, 0.001),
                                                     (V2A, 4, 24700, 10752, 48, 0.001), (V2A, 2, 24577, 8320, 40, 0.0), (V2, 3, 24577, 8320, 33, None)])
def test_long_rows_and_matrices_without_outliers(mode, bits, N, K, M, density):
    W = xi.random_weights(mode, bits, N, K, density=density or 0.0, seed=N + K)
    if density is None:
        W.out_row_ptr = np.concatenate([np.zeros(N, np.int32), np.array([9], np.int32)])
        W.out_col, W.out_val = np.arange(0, K, K // 9, dtype=np.int32)[:9], xi.activations(np.random.default_rng(2), 1, 9).ravel()
    x = xi.activations(np.random.default_rng(K + M), M, K)
    dW, xd = xfp.upload(W), torch.from_numpy(x.view(np.int16)).cuda().view(torch.float16)
    assert xfp.xfp_launch_route(dW, M) == (xfp.XFP_ROUTE_WIDE, M) and xfp.xfp_wide_tile(dW, M) == TILE(M)
    y = xfp.xfp_gemv(dW, xd, y_dtype=torch.float32)
    rows = np.unique(np.concatenate([np.arange(0, N, 997), np.arange(N - 140, N)]))                        # (the oracle's time)
    assert gated_rel_err(y.cpu().numpy()[:, rows].astype(np.float64), oracle.gemv_weights(some_rows(W, rows), x)) <= 1e-4


def some_rows(W, rows):
    ptr = W.out_row_ptr
    pick = np.concatenate([np.arange(ptr[r], ptr[r + 1]) for r in rows] + [np.zeros(0, np.int64)]).astype(np.int64)
    V = copy.copy(W)
    V.N, V.indices = len(rows), W.indices[:, rows]
    if W.mode == V2:
        V.codebooks = W.codebooks[:, rows]
    else:
        V.group_ids = W.group_ids[:, rows]
    V.out_row_ptr = np.concatenate([[0], np.cumsum([ptr[r + 1] - ptr[r] for r in rows])]).astype(np.int32)
    V.out_col, V.out_val = W.out_col[pick], W.out_val[pick]
    return V


@pytest.mark.parametrize("mode,bits,M", [(V2, 4, 30), (V2A, 3, 50)])
def test_bf16_strides_and_untouched_padding(mode, bits, M):
    N, K = 24700, 1664
    W = xi.random_weights(mode, bits, N, K, density=0.003, seed=M)
    x = torch.randn((M, K + 24), device="cuda").bfloat16()[:, :K]
    dW = xfp.upload(W)
    assert xfp.xfp_launch_route(dW, M) == (xfp.XFP_ROUTE_WIDE, M) and xfp.xfp_wide_tile(dW, M) == TILE(M)
    want = xfp.xfp_gemv(dW, xfp.xfp_convert_bf16_to_f16(x), y_dtype=torch.float32)
    for ldy in (N + 3, N + 4):                                                             # single and four-value stores
        buf = torch.full((M, ldy), -3.0, dtype=torch.bfloat16, device="cuda")
        xfp.xfp_gemv(dW, x, y=buf[:, :N])
        assert torch.equal(buf[:, :N], want.bfloat16()) and bool((buf[:, N:] == -3.0).all())


@pytest.mark.parametrize("M", [29, 64])
def test_infinities_and_nan_stay_with_their_tokens(M):
    W = xi.random_weights(V2, 3, 24600, 1920, density=0.01, seed=M)
    x, dW = torch.randn(M, W.K, device="cuda").half(), xfp.upload(W)
    assert xfp.xfp_launch_route(dW, M) == (xfp.XFP_ROUTE_WIDE, M) and xfp.xfp_wide_tile(dW, M) == TILE(M)
    clean = xfp.xfp_gemv(dW, x, y_dtype=torch.float32)
    x[3, 7], x[M - 1, W.K - 1] = float("inf"), float("nan")
    y = xfp.xfp_gemv(dW, x, y_dtype=torch.float32)
    rest = [m for m in range(M) if m not in (3, M - 1)]
    assert torch.equal(y[rest], clean[rest]) and torch.isnan(y[M - 1]).all() and not torch.isfinite(y[3]).any()


def test_they_replay_from_a_graph():
    W = xi.random_weights(V2A, 4, 24600, 1664, density=0.003, seed=7)
    dW, x = xfp.upload(W), torch.randn(30, W.K, device="cuda").half()
    assert xfp.xfp_launch_route(dW, 30) == (xfp.XFP_ROUTE_WIDE, 30) and xfp.xfp_wide_tile(dW, 30) == TILE(30)
    xfp.xfp_gemv(dW, x, y_dtype=torch.float32)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        y = xfp.xfp_gemv(dW, x, y_dtype=torch.float32)
    for i in range(4):
        x.copy_(torch.randn(30, W.K, device="cuda").half())
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, xfp.xfp_gemv(dW, x, y_dtype=torch.float32))
