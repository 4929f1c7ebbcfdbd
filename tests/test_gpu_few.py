"""The kernel that keeps the activations in LDS (2 to 64 tokens, one launch; xfp_decode_few): parity with the oracle at the
edges of its blocks, units, slices and outlier windows, non-finite activations, other types, graph replay."""
import numpy as np
import pytest
import torch

import oracle
import paper_2605_14844_amd as xfp
import xfp_inputs as xi
from helpers import gated_rel_err

pytestmark = pytest.mark.gpu
V2, V2A = xi.MODE_V2, xi.MODE_V2A


def dev_x(x_bits):
    return torch.from_numpy(np.ascontiguousarray(x_bits).view(np.int16)).cuda().view(torch.float16)


def host(y):
    torch.cuda.synchronize()
    return y.float().cpu().numpy().astype(np.float64)


def with_records(W, seed):
    r = np.random.default_rng(seed)
    n = (W.E, W.N, W.K // 128)
    W.group_scale = (r.random(n) * 0.5 + 0.5).astype(np.float16).view(np.uint16)
    W.group_mid = (r.standard_normal(n) * 0.01).astype(np.float16).view(np.uint16)
    return W


def check(W, x):
    ref = oracle.gemv_weights(W, x)
    y = xfp.xfp_gemv(xfp.upload(W), dev_x(x), y_dtype=torch.float32)
    err = gated_rel_err(host(y), ref)
    print(f"  N={W.N} K={W.K} M={x.shape[0]}: {err:.2e}", flush=True)
    assert err <= 1e-4                                                # fp32 results, as in the other kernels' tests
    return y


# one group; rows that fill no block and tokens that fill no chunk; an odd number of groups (half a unit at 2 bits); fewer
# units than waves; more blocks than CUs; 32 and 64 tokens; several slices with a shorter last one (10880, 14336 columns)
SIZES = [(16, 128, 2), (1, 128, 16), (33, 384, 3), (250, 640, 7), (77, 1152, 16), (4100, 256, 9), (9000, 1408, 2),
         (300, 2048, 17), (300, 1536, 32), (300, 4096, 33), (200, 8320, 64), (130, 10880, 12), (70, 14336, 41)]


@pytest.mark.parametrize("N,K,M", SIZES)
@pytest.mark.parametrize("bits", [4, 3, 2])
@pytest.mark.parametrize("mode", [V2, V2A, 2])
def test_resident_kernel_matches_oracle(mode, bits, N, K, M):
    W = xi.random_weights(V2A if mode == 2 else mode, bits, N, K, density=0.01 if K <= 2048 else 0.003, seed=N + K + M)
    if mode == 2:
        with_records(W, K)
    check(W, xi.activations(np.random.default_rng(M + N), M, K))


# 5 and 6 bits (tables of one entry per index): rows that fill no block, one group, more outliers than pass through LDS at
# once, several passes of fewer tokens because the activations do not fit; the last two stay in the general kernel
@pytest.mark.parametrize("N,K,M,density", [(4097, 128, 2, 0.01), (4100, 256, 17, 0.01), (5003, 1408, 5, 0.05), (9000, 384, 64, 0.003),
                                           (70, 14336, 43, 0.003), (4111, 8320, 21, 0.001), (333, 1152, 13, 0.01), (4097, 512, 1, 0.01)])
@pytest.mark.parametrize("bits", [5, 6])
def test_wide_indices_match_oracle(bits, N, K, M, density):
    check(xi.random_weights(V2, bits, N, K, density=density, seed=N + M), xi.activations(np.random.default_rng(M), M, K))


def test_large_libraries_and_one_token_of_long_library_rows():
    check(xi.random_weights(V2A, 4, 100, 1280, L=256, density=0.003, seed=1), xi.activations(np.random.default_rng(1), 5, 1280))
    check(xi.random_weights(V2A, 2, 4100, 16512, L=3, density=0.001, seed=2), xi.activations(np.random.default_rng(2), 1, 16512))


@pytest.mark.parametrize("mode,bits,N", [(V2, 2, 300), (V2A, 3, 33), (V2A, 4, 2050), (2, 2, 2049), (V2, 4, 100)])
def test_one_token_of_rows_without_equal_slices(mode, bits, N):
    """139 groups: no number of equal slices is short enough for the streaming kernel (the last stays in the general kernel)."""
    W = xi.random_weights(V2A if mode == 2 else mode, bits, N, 139 * 128, density=0.003, seed=N)
    check(with_records(W, 3) if mode == 2 else W, xi.activations(np.random.default_rng(N), 1, W.K))


@pytest.mark.parametrize("M", [2, 16, 40])
def test_rows_with_more_outliers_than_pass_through_lds_at_once(M):
    """One row holds 700 entries (three windows of 256), the next none, its neighbours a few: windows move within a row, and
    go back for the next 16 tokens."""
    W = xi.random_weights(V2, 4, 48, 2048, density=0.0, seed=9)
    counts = np.zeros(48, np.int64)
    counts[17], counts[16], counts[19], counts[47] = 700, 3, 300, 40
    r = np.random.default_rng(1)
    W.out_row_ptr = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    W.out_col = np.concatenate([np.sort(r.choice(W.K, size=c, replace=False)) for c in counts]).astype(np.int32)
    W.out_val = xi.activations(np.random.default_rng(2), 1, int(counts.sum())).ravel()
    check(W, xi.activations(np.random.default_rng(3), M, W.K))


@pytest.mark.parametrize("mode,N,K,M", [(V2A, 4100, 28672, 1), (V2A, 33, 28672, 2), (V2, 50, 16640, 3), (V2, 20, 9088, 5), (V2, 20, 128, 2)])
def test_outliers_of_token_counts_that_are_no_multiple_of_four(mode, N, K, M):
    """An entry's activations are read four tokens at a time; rows as long as a workgroup's LDS, infinities in the last token."""
    W = xi.random_weights(mode, 3, N, K, density=0.01, seed=N + M)
    x = xi.activations(np.random.default_rng(K), M, K)
    y = check(W, x)
    x[M - 1, ::7] = 0x7C00                                            # (V2A entries and outliers of both signs: no finite result)
    special = xfp.xfp_gemv(xfp.upload(W), dev_x(x), y_dtype=torch.float32)
    assert torch.equal(special[:M - 1], y[:M - 1]) and not torch.isfinite(special[M - 1]).any()


@pytest.mark.parametrize("K", [1152, 10880])
def test_infinities_and_nan_stay_with_their_tokens(K):
    W = xi.random_weights(V2A, 2, 50, K, density=0.01, seed=4)
    x = dev_x(xi.activations(np.random.default_rng(5), 13, K))
    dW = xfp.upload(W)
    clean = xfp.xfp_gemv(dW, x, y_dtype=torch.float32)
    x[3, 7], x[12, K - 1], x[0, 0] = float("inf"), float("nan"), float("-inf")
    y = xfp.xfp_gemv(dW, x, y_dtype=torch.float32)
    for m in range(13):
        if m in (0, 3, 12):
            assert not torch.isfinite(y[m]).any()
        else:
            assert torch.equal(y[m], clean[m])


def test_types_strides_and_repeats():
    """bf16 activations give what the converted ones give; padded rows of x and y; 16-bit results are the fp32 ones, rounded;
    the entry point that allocates nothing agrees; results repeat bit for bit."""
    W = xi.random_weights(V2, 3, 333, 2176, density=0.003, seed=6)
    dW = xfp.upload(W)
    wide = torch.randn((9, 2176 + 24), device="cuda").to(torch.bfloat16)
    xb = wide[:, :2176]
    y = xfp.xfp_gemv(dW, xb, y_dtype=torch.float32)
    assert torch.equal(y, xfp.xfp_gemv(dW, xb.half(), y_dtype=torch.float32))
    assert torch.equal(y.half(), xfp.xfp_gemv(dW, xb, y_dtype=torch.float16))
    assert torch.equal(y.bfloat16(), xfp.xfp_gemv(dW, xb, y_dtype=torch.bfloat16))
    out = torch.full((9, 340), 7.0, device="cuda")
    xfp.xfp_gemv_noalloc(dW, xb, out[:, :333])
    assert torch.equal(out[:, :333], y) and bool((out[:, 333:] == 7.0).all())
    for _ in range(5):
        assert torch.equal(xfp.xfp_gemv(dW, xb, y_dtype=torch.float32), y)


@pytest.mark.parametrize("K", [1024, 12288])
def test_graph_replays_match_eager_calls(K):
    W = xi.random_weights(V2, 4, 100, K, density=0.003, seed=7)
    dW, x = xfp.upload(W), dev_x(xi.activations(np.random.default_rng(8), 14, K))
    xfp.xfp_gemv(dW, x, y_dtype=torch.float32)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        y = xfp.xfp_gemv(dW, x, y_dtype=torch.float32)
    for i in range(4):
        x.copy_(dev_x(xi.activations(np.random.default_rng(20 + i), 14, K)))
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, xfp.xfp_gemv(dW, x, y_dtype=torch.float32))
