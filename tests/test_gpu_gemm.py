"""The prompt kernel (many tokens as one tiled product, V2 and V2a at 2 to 4 bits): parity with the oracle at the
edges of its tiles, its order of k bit-exactly through one-hot activations, types, strides and repeatability."""
import os
import re
import subprocess
import sys

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


# N: the fewest rows, a ragged last row tile, one row more than a tile; K: one group (fewer columns than a stage of
# the small tile), odd group counts, a row of 64 groups; M: the fewest tokens that it is preferred for, ragged last
# token tiles, more than a tile; outliers: none, the benchmark's density, more than LDS holds of a tile
@pytest.mark.parametrize("N,K,M,dens", [(128, 128, 193, 0.01), (129, 384, 257, 0.003), (200, 4096, 200, 0.003), (257, 1152, 333, 0.0),
                                        (128, 8192, 198, 0.04), (8200, 256, 1500, 0.003), (8193, 640, 1537, 0.002)])
@pytest.mark.parametrize("bits", [4, 3, 2])
@pytest.mark.parametrize("mode", [V2, V2A])
def test_prompt_parity(mode, bits, N, K, M, dens):
    W = xi.random_weights(mode, bits, N, K, L=33, density=dens, seed=N + K + M + bits)
    xb = xi.activations(np.random.default_rng(M), M, K)
    dW, xd = xfp.upload(W), dev_x(xb)
    assert xfp.xfp_route(dW, M) == (xfp.XFP_ROUTE_GEMM, M)
    y32, y16 = xfp.xfp_gemv(dW, xd, y_dtype=torch.float32), xfp.xfp_gemv(dW, xd)
    again = xfp.xfp_gemv(dW, xd, y_dtype=torch.float32)
    torch.cuda.synchronize()
    ref = oracle.gemv_weights(W, xb)
    assert gated_rel_err(y32.cpu().numpy(), ref) <= 1e-4
    assert gated_rel_err(y16.float().cpu().numpy(), ref) <= 1e-3
    assert torch.equal(y32, again)


# rows of a block or two, which have tiles of their own (up to 512 columns of 64 x 64 tiles, 256 of 128 x 64): both sides of either
# limit, ragged last tiles, waves with no block, an infinity and a NaN that stay with their tokens
@pytest.mark.parametrize("N,K,M", [(130, 128, 95), (143, 256, 150), (700, 384, 97), (212, 512, 92), (213, 640, 92), (8193, 128, 130), (6145, 256, 200), (8300, 384, 131)])
@pytest.mark.parametrize("mode,bits", [(V2, 4), (V2A, 3), (V2, 2), (V2A, 4), (V2, 3), (V2A, 2)])
def test_short_rows(mode, bits, N, K, M):
    W = xi.random_weights(mode, bits, N, K, L=33, density=0.01, seed=N + K + M + bits)
    xb = xi.activations(np.random.default_rng(M), M, K)
    dW, xd = xfp.upload(W), dev_x(xb)
    assert xfp.xfp_launch_route(dW, M) == (xfp.XFP_ROUTE_GEMM, M)
    y = xfp.xfp_gemv(dW, xd, y_dtype=torch.float32)
    assert gated_rel_err(y.cpu().numpy(), oracle.gemv_weights(W, xb)) <= 1e-4
    assert torch.equal(xfp.xfp_gemv(dW, xd), y.half())
    xd[3, 7], xd[M - 1, K - 1] = float("inf"), float("nan")
    z = xfp.xfp_gemv(dW, xd, y_dtype=torch.float32)
    rest = [m for m in range(M) if m not in (3, M - 1)]
    assert torch.equal(z[rest], y[rest]) and torch.isnan(z[M - 1]).all() and not torch.isfinite(z[3]).any()


@pytest.mark.parametrize("mode,bits,K", [(V2, 4, 640), (V2, 3, 640), (V2, 2, 384), (V2A, 4, 384), (V2A, 3, 640), (V2A, 2, 384)])
def test_one_hot_tokens_read_single_weights(mode, bits, K):
    """Token m is one at column (7 m) mod K: y[m][n] is that column of the matrix, one rounding of the sum of its codebook
    entry and (where there is one) its outlier."""
    W = xi.random_weights(mode, bits, 150, K, L=5, density=0.02, seed=bits)
    M = K + 3
    cols = (7 * np.arange(M)) % K
    x = np.zeros((M, K), dtype=np.float16)
    x[np.arange(M), cols] = 1.0
    dW = xfp.upload(W)
    y = xfp.xfp_gemv(dW, torch.from_numpy(x).cuda(), y_dtype=torch.float32)
    bulk = xfp.xfp_dequant_bulk(dW).view(torch.float16).float()
    torch.cuda.synchronize()
    dense = bulk.cpu().numpy()
    for n in range(W.N):
        s = slice(W.out_row_ptr[n], W.out_row_ptr[n + 1])
        dense[n, W.out_col[s]] += W.out_val[s].view(np.float16).astype(np.float32)
    assert np.array_equal(y.cpu().numpy(), dense.T[cols])


@pytest.mark.parametrize("N,M", [(300, 228), (8196, 1600)])
def test_bf16_strides_and_untouched_padding(N, M):
    K = 512
    W = xi.random_weights(V2, 4, N, K, density=0.003, seed=77)
    x = torch.randn((M, K + 24), generator=torch.Generator().manual_seed(3)).bfloat16()
    x = torch.where(x.abs() < 2.0 ** -10, torch.full_like(x, 0.5), x)                       # exact in fp16
    ref = oracle.gemv_weights(W, x[:, :K].half().contiguous().view(torch.int16).numpy().view(np.uint16))
    dW = xfp.upload(W)
    for ldy in (N + 3, N + 4):                                                             # single and four-value stores
        buf = torch.full((M, ldy), -3.0, dtype=torch.bfloat16, device="cuda")
        xfp.xfp_gemv(dW, x.cuda()[:, :K], y=buf[:, :N])
        torch.cuda.synchronize()
        assert gated_rel_err(buf[:, :N].float().cpu().numpy(), ref) <= 6e-3
        assert torch.all(buf[:, N:] == -3.0)


# 28672 x 585 and 24576 x 682: one token more than a multiple of 8 that both copies hold (2^24 halves each: a row of the
# k-major one is the tokens rounded up to 8); 65536 columns: 256 tokens a launch, none left for the kernels of few tokens
@pytest.mark.parametrize("bits,N,K,M,dens,first", [(4, 130, 28672, 585, 0.002, 512), (3, 140, 24576, 682, 0.002, 512), (2, 130, 24576, 680, 0.002, 680),
                                                   (2, 130, 65536, 256 + 37, 0.001, 152), (4, 140, 5120, 3273, 0.002, 3072)])
def test_more_tokens_than_the_copies_hold(bits, N, K, M, dens, first):
    W = xi.random_weights(V2, bits, N, K, density=dens, seed=5)
    xb = xi.activations(np.random.default_rng(9), M, K)
    dW = xfp.upload(W)
    assert xfp.xfp_route(dW, M) == (xfp.XFP_ROUTE_GEMM, first)
    y = xfp.xfp_gemv(dW, dev_x(xb), y_dtype=torch.float32)
    torch.cuda.synchronize()
    assert gated_rel_err(y.cpu().numpy(), oracle.gemv_weights(W, xb)) <= 1e-4


# 128 x 64 tiles (16 waves at 2 bits) and 256 x 128 tiles; rows whose chains are half a block, rows on either side of that,
# rows with a third set of sums
@pytest.mark.parametrize("bits,N,K,M,mode", [(4, 1024, 512, 520, V2), (2, 1024, 1536, 520, V2A), (3, 1024, 3072, 520, V2), (2, 1024, 4096, 520, V2A), (4, 1024, 8192, 520, V2),
                                             (3, 1024, 28672, 520, V2), (2, 1024, 28672, 520, V2), (4, 8320, 512, 520, V2), (3, 8320, 2048, 520, V2A),
                                             (4, 8320, 3072, 520, V2), (4, 8320, 8192, 520, V2)])
@pytest.mark.parametrize("dens", [0.0, 0.003])
def test_sums_are_as_exact_as_in_passes_of_64_tokens(bits, N, K, M, mode, dens):
    """Against 64 bits, the fp32 results are no further off than those of the same tokens in passes of 64 (5 % for what two
    samples of half a million rounding errors differ by); 16-bit results are the fp32 results, rounded."""
    W = xi.random_weights(mode, bits, N, K, L=16, density=dens, seed=K + bits)
    x = dev_x(xi.activations(np.random.default_rng(K), M, K))
    dW = xfp.upload(W)
    assert xfp.xfp_route(dW, M) == (xfp.XFP_ROUTE_GEMM, M) and xfp.xfp_route(dW, 64)[0] != xfp.XFP_ROUTE_GEMM
    dense = xfp.xfp_dequant_bulk(dW).view(torch.float16).double()
    ptr = torch.from_numpy(W.out_row_ptr.astype(np.int64)).cuda()
    rows = torch.repeat_interleave(torch.arange(N, device="cuda"), ptr[1:] - ptr[:-1])
    dense[rows, torch.from_numpy(W.out_col.astype(np.int64)).cuda()] += torch.from_numpy(W.out_val.view(np.float16).astype(np.float64)).cuda()
    exact = x.double() @ dense.T
    y = xfp.xfp_gemv(dW, x, y_dtype=torch.float32)
    passes = torch.cat([xfp.xfp_gemv(dW, x[i:i + 64], y_dtype=torch.float32) for i in range(0, M, 64)])
    err = [float(((v.double() - exact).norm() / exact.norm()).item()) for v in (y, passes)]
    assert err[0] <= 1.05 * err[1], err
    for t in (torch.float16, torch.bfloat16):
        assert torch.equal(xfp.xfp_gemv(dW, x, y_dtype=t), y.to(t))


@pytest.mark.parametrize("bits,L", [(4, 256), (3, 255), (2, 256)])
def test_the_largest_libraries(bits, L):
    """No other matrix-core kernel takes them; every entry is used, the last one too."""
    W = xi.random_weights(V2A, bits, 300, 896, L=L, density=0.003, seed=L + bits)
    W.group_ids.reshape(-1)[:L] = np.arange(L, dtype=np.uint8)
    xb = xi.activations(np.random.default_rng(L), 230, 896)
    dW = xfp.upload(W)
    assert xfp.xfp_route(dW, 230) == (xfp.XFP_ROUTE_GEMM, 230)
    y = xfp.xfp_gemv(dW, dev_x(xb), y_dtype=torch.float32)
    torch.cuda.synchronize()
    assert gated_rel_err(y.cpu().numpy(), oracle.gemv_weights(W, xb)) <= 1e-4


# odd group counts (half a block is zero times zero), one and several tiles of rows, 64 x 64 and 256 x 128 tiles
@pytest.mark.parametrize("bits,N,K,M,mode", [(4, 200, 384, 200, V2), (3, 130, 640, 200, V2A), (2, 130, 896, 200, V2), (2, 8200, 640, 600, V2)])
def test_infinities_and_nan_stay_with_their_tokens(bits, N, K, M, mode):
    W = xi.random_weights(mode, bits, N, K, L=9, density=0.01, seed=N + bits)
    x = dev_x(xi.activations(np.random.default_rng(M), M, K)).clone()
    dW = xfp.upload(W)
    assert xfp.xfp_route(dW, M) == (xfp.XFP_ROUTE_GEMM, M)
    plain = xfp.xfp_gemv(dW, x, y_dtype=torch.float32)
    special = {3: (K - 1, np.inf), 64: (0, -np.inf), M - 1: (K // 2, np.nan)}
    for m, (k, v) in special.items():
        x[m, k] = v
    y = xfp.xfp_gemv(dW, x, y_dtype=torch.float32).cpu().numpy()
    weight = xfp.xfp_dequant_bulk(dW).view(torch.float16).float().cpu().numpy()
    for m, (k, v) in special.items():
        with np.errstate(invalid="ignore"):
            want = weight[:, k] * np.float32(v)
            for n in range(N):
                at = np.flatnonzero(W.out_col[W.out_row_ptr[n]:W.out_row_ptr[n + 1]] == k)
                for j in at:
                    want[n] += np.float32(W.out_val[W.out_row_ptr[n] + j].view(np.float16)) * np.float32(v)
        assert np.array_equal(y[m], want, equal_nan=True), m
    rest = [m for m in range(M) if m not in special]
    assert np.array_equal(y[rest], plain.cpu().numpy()[rest])


FIRST_PROMPT = """
import sys
import numpy as np, torch
import paper_2605_14844_amd as xfp, xfp_inputs as xi

def used():
    torch.cuda.synchronize()
    free, total = torch.cuda.mem_get_info()
    return (total - free) >> 20

W = xfp.upload(xi.random_weights(xi.MODE_V2, 4, 256, 512, density=0.003, seed=3))
M = int(sys.argv[1])
x = torch.from_numpy(xi.activations(np.random.default_rng(4), M, 512).view(np.int16)).cuda().view(torch.float16)
y, y4 = torch.empty((M, 256), dtype=torch.float16, device="cuda"), torch.empty((4, 256), dtype=torch.float16, device="cuda")
xfp.xfp_gemv(W, x[:1], y=y4[:1])
before = used()
xfp.xfp_init()
xfp.xfp_gemv(W, x[:4], y=y4)
xfp.xfp_gemv_noalloc(W, x[:4], y4)
few = used() - before
side, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
with torch.cuda.graph(graph, stream=side):
    xfp.xfp_gemv(W, x, y=y)
prompt = used() - before
seen = []
for _ in range(3):
    y.zero_()
    graph.replay()
    torch.cuda.synchronize()
    seen.append(y.clone())
    xfp.xfp_gemv(W, x[:4], y=y4)
eager, fixed = xfp.xfp_gemv(W, x), torch.empty_like(y)
xfp.xfp_gemv_noalloc(W, x, fixed)
torch.cuda.synchronize()
assert all(torch.equal(s, eager) for s in seen) and torch.equal(fixed, eager)
print("MB", few, prompt, used() - before)
"""


@pytest.mark.parametrize("M", [600, 100])
def test_only_prompts_load_the_memory_of_prompts(M):
    """Eight workspaces and the static array are 90 MB; the first tiled product, of a prompt or of a batch of more than 64 tokens,
    loads 512 more (and 64 for xfp_gemv_noalloc), also where it is a call that is being captured."""
    r = subprocess.run([sys.executable, "-c", FIRST_PROMPT, str(M)], cwd=os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                       capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stderr[-2000:]
    few, prompt, both = map(int, re.search(r"MB (\d+) (\d+) (\d+)", r.stdout).groups())
    assert few <= 130 and 512 <= prompt - few and 64 <= both - prompt and both <= 760, (few, prompt, both)
