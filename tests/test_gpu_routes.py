"""Every kernel for several tokens at shapes that the dispatch sends to it (asserted through xfp_launch_route): the 16-token, the
64-token and the prompt kernel where the resident kernel does not take the call.  Parity with the oracle; for the resident kernel
how exact its sums are beside the kernels that it stands in for."""
import numpy as np
import pytest
import torch

import oracle
import paper_2605_14844_amd as xfp
import xfp_inputs as xi
from helpers import gated_rel_err

pytestmark = pytest.mark.gpu
V2, V2A = xi.MODE_V2, xi.MODE_V2A
BATCH, WIDE, GEMM, RESIDENT = xfp.XFP_ROUTE_BATCH, xfp.XFP_ROUTE_WIDE, xfp.XFP_ROUTE_GEMM, xfp.XFP_ROUTE_RESIDENT


def dev_x(x_bits):
    return torch.from_numpy(np.ascontiguousarray(x_bits).view(np.int16)).cuda().view(torch.float16)


def host(y):
    torch.cuda.synchronize()
    return y.float().cpu().numpy().astype(np.float64)


def launches(dW, M):
    out = []
    while M:
        out.append(xfp.xfp_launch_route(dW, M))
        M -= out[-1][1]
    return out


def check(W, M, first, seed=0):
    """fp32, fp16 and bf16 results against the oracle, and the call that allocates nothing; first: the call's first launch"""
    x = xi.activations(np.random.default_rng(W.N + W.K + M + seed), M, W.K)
    dW, xd, ref = xfp.upload(W), dev_x(x), oracle.gemv_weights(W, x)
    assert launches(dW, M)[0] == first, launches(dW, M)
    y = xfp.xfp_gemv(dW, xd, y_dtype=torch.float32)
    err = gated_rel_err(host(y), ref)
    print(f"  mode={W.mode} bits={W.bits} N={W.N} K={W.K} M={M} {launches(dW, M)}: {err:.2e}", flush=True)
    assert err <= 1e-4                                                # fp32 results, as in the other kernels' tests
    for t in (torch.float16, torch.bfloat16):
        assert torch.equal(xfp.xfp_gemv(dW, xd, y_dtype=t), y.to(t))
    fixed = torch.full((M, W.N), 7.0, device="cuda")
    xfp.xfp_gemv_noalloc(dW, xd, fixed)
    assert torch.equal(fixed, y)
    return dW, xd, y


# ---------------------------------------------------------------- the 16-token kernel
# groups per wave 3 to 8, with and without a short last wave; sixteen tokens, one token row of a tile, ragged tiles
@pytest.mark.parametrize("mode,bits,N,K,M", [(V2, 4, 50000, 3072, 16), (V2A, 3, 50000, 2944, 16), (V2, 3, 33000, 4096, 16), (V2A, 4, 33001, 3712, 16),
                                             (V2, 2, 33000, 5120, 16), (V2A, 2, 32800, 4736, 16), (V2, 4, 7100, 6144, 16), (V2A, 3, 7109, 6016, 16),
                                             (V2, 2, 9001, 5760, 16), (V2A, 2, 4200, 6784, 16), (V2, 3, 2100, 7168, 14), (V2A, 4, 2107, 6272, 16),
                                             (V2, 4, 1, 8192, 16), (V2, 3, 40, 8064, 16), (V2A, 4, 33, 8192, 16), (V2A, 3, 17, 8064, 16),
                                             (V2, 2, 2100, 7808, 16), (V2A, 2, 2050, 8192, 16)])
def test_16_token_kernel(mode, bits, N, K, M):
    check(xi.random_weights(mode, bits, N, K, density=0.001 if N > 9000 else 0.003, seed=N + K), M, (BATCH, M))


# slices of 48, 56 and 64 groups, the last one shorter, and of 40 nowhere; the token behind the sixteen
@pytest.mark.parametrize("mode,bits,N,K,M", [(V2, 4, 1009, 16512, 17), (V2A, 3, 1010, 18560, 17), (V2, 2, 1009, 21632, 17), (V2A, 4, 1023, 20480, 18),
                                             (V2, 3, 3000, 28672, 16), (V2A, 2, 1009, 32768, 17)])
def test_16_token_kernel_in_slices(mode, bits, N, K, M):
    check(xi.random_weights(mode, bits, N, K, density=0.002, seed=N + K), M, (BATCH, 16))


@pytest.mark.parametrize("bits,L", [(4, 64), (3, 200), (3, 1), (4, 7), (2, 256), (2, 3)])
def test_16_token_kernel_library_sizes(bits, L):
    check(xi.random_weights(V2A, bits, 2100 if bits == 2 else 70, 8192, L=L, density=0.003, seed=L), 16, (BATCH, 16))


def test_16_token_kernel_with_more_outliers_than_a_tile_keeps_on_chip():
    check(xi.random_weights(V2, 4, 80, 8192, density=0.05, seed=77), 16, (BATCH, 16))
    K = 8192
    W = xi.random_weights(V2, 4, 40, K, density=0.0, seed=78)
    rp = np.zeros(41, dtype=np.int32)
    rp[18:] = K                                                       # row 17 holds all K entries
    W.out_row_ptr, W.out_col = rp, np.arange(K, dtype=np.int32)
    W.out_val = xi.activations(np.random.default_rng(71), 1, K).ravel()
    x = xi.activations(np.random.default_rng(72), 16, K)
    dW = xfp.upload(W)
    assert xfp.xfp_launch_route(dW, 16) == (BATCH, 16)
    y, ref = host(xfp.xfp_gemv(dW, dev_x(x), y_dtype=torch.float32)), oracle.gemv_weights(W, x)
    # a sum of n terms of random sign in one fp32 chain is off by 2^-24 sqrt(n / 2) of its size
    for r in (np.arange(40) == 17, np.arange(40) != 17):
        assert np.linalg.norm(y[:, r] - ref[:, r]) <= 2.0 ** -24 * (K / 2) ** 0.5 * np.linalg.norm(ref[:, r])


# ---------------------------------------------------------------- the 64-token kernel
# one chunk (long rows of tall matrices), two, three and four; the longest row of each; dense outliers
@pytest.mark.parametrize("mode,bits,N,K,M,first", [(V2, 4, 8161, 11008, 9, 9), (V2A, 3, 8170, 8320, 12, 12), (V2, 2, 8161, 8320, 16, 16), (V2, 3, 8161, 28672, 9, 9),
                                                   (V2, 4, 1009, 2304, 32, 32), (V2A, 2, 1020, 2688, 25, 25), (V2, 3, 1009, 16384, 32, 32), (V2A, 4, 1100, 4096, 31, 31),
                                                   (V2, 2, 1009, 10880, 47, 47), (V2A, 3, 1013, 10880, 48, 48), (V2, 4, 641, 8064, 64, 64), (V2A, 4, 700, 4096, 49, 49)])
def test_64_token_kernel(mode, bits, N, K, M, first):
    check(xi.random_weights(mode, bits, N, K, density=0.01 if K < 4096 else 0.002, seed=N + K), M, (WIDE, first))


# a scale and a mid-point per group: chunks of 16; ragged last tile, the shortest and the longest rows that reach it, large libraries
@pytest.mark.parametrize("bits,N,K,M,L", [(3, 1100, 7808, 16, 32), (4, 1101, 8192, 16, 60), (2, 1009, 8320, 17, 7), (3, 8200, 12288, 16, 200), (4, 1010, 32768, 40, 1),
                                          (2, 8193, 8192, 40, 256)])
def test_64_token_kernel_with_records(bits, N, K, M, L):
    W = xi.random_weights(V2A, bits, N, K, L=L, density=0.002, seed=N + K + bits, affine=True)
    dW, xd, y = check(W, M, (WIDE, 16))
    xb = xd.float().bfloat16()                                        # bf16 activations: the converted call's bits
    assert torch.equal(xfp.xfp_gemv(dW, xb, y_dtype=torch.float32), xfp.xfp_gemv(dW, xfp.xfp_convert_bf16_to_f16(xb), y_dtype=torch.float32))


def test_64_token_kernel_one_hot_is_the_affine_value():
    """y[m][n] = entry * scale + mid of one weight: one fp32 rounding of an exact product plus the mid-point."""
    W = xi.random_weights(V2A, 4, 1100, 8192, L=9, density=0.0, seed=10, affine=True)
    dW = xfp.upload(W)
    assert xfp.xfp_launch_route(dW, 16) == (WIDE, 16)
    q = oracle.unpack(W.indices[0], W.K, 4).astype(np.int64)
    lib = W.codebooks[0].view(np.float16).astype(np.float64)
    ids, sc, md = (np.repeat(v, 128, axis=1) for v in (W.group_ids[0].astype(np.int64), W.group_scale[0].view(np.float16).astype(np.float64),
                                                       W.group_mid[0].view(np.float16).astype(np.float64)))
    want = (lib[ids, q] * sc + md).astype(np.float32)
    for k0 in (0, 500, 8176):
        x = np.zeros((16, W.K), np.float16)
        x[np.arange(16), k0 + np.arange(16)] = 1.0
        got = xfp.xfp_gemv(dW, dev_x(x.view(np.uint16)), y_dtype=torch.float32).cpu().numpy()
        assert np.array_equal(got, want[:, k0:k0 + 16].T)


# ---------------------------------------------------------------- the tiled product below 193 tokens and beyond a round of tiles
# both sides of every limit of its rule: 80 tokens, 65 of long rows, 128 of few long rows; a little more than a round of tiles;
# a pass and a round; several launches
@pytest.mark.parametrize("mode,bits,N,K,M,first", [
    (V2, 4, 1200, 4096, 80, (GEMM, 80)), (V2, 4, 1200, 4096, 79, (WIDE, 64)), (V2A, 2, 129, 640, 81, (GEMM, 81)), (V2A, 3, 1030, 8192, 80, (GEMM, 80)),
    (V2, 3, 2048, 8320, 65, (GEMM, 65)), (V2A, 4, 2050, 8320, 66, (GEMM, 66)), (V2, 2, 2047, 8320, 79, (WIDE, 48)), (V2, 2, 600, 8192, 128, (GEMM, 128)),
    (V2A, 4, 600, 8192, 127, (RESIDENT, 64)), (V2, 4, 1300, 5120, 192, (GEMM, 192)), (V2, 4, 1300, 5120, 193, (GEMM, 193)),
    (V2A, 3, 11100, 3072, 129, (WIDE, 64)), (V2, 2, 11100, 1152, 161, (GEMM, 161)), (V2, 4, 8192, 2176, 320, (WIDE, 64)), (V2, 3, 12300, 640, 257, (GEMM, 257)),
    (V2, 4, 130, 28672, 586, (GEMM, 512))])
def test_tiled_product_of_few_tokens(mode, bits, N, K, M, first):
    check(xi.random_weights(mode, bits, N, K, density=0.002, seed=N + K), M, first)


def test_tiled_product_of_few_tokens_replays_from_a_graph():
    W = xi.random_weights(V2A, 3, 300, 2176, density=0.003, seed=7)
    dW, x = xfp.upload(W), dev_x(xi.activations(np.random.default_rng(8), 100, W.K))
    assert xfp.xfp_launch_route(dW, 100) == (GEMM, 100)
    xfp.xfp_gemv(dW, x, y_dtype=torch.float32)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        y = xfp.xfp_gemv(dW, x, y_dtype=torch.float32)
    for i in range(4):
        x.copy_(dev_x(xi.activations(np.random.default_rng(20 + i), 100, W.K)))
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, xfp.xfp_gemv(dW, x, y_dtype=torch.float32))


# ---------------------------------------------------------------- the resident kernel
# waves without a unit (rows of one to three), slices in one round of the CUs (three of 4 blocks, eight of 8), 5 and 6 bits
@pytest.mark.parametrize("mode,bits,N,K,M", [(V2, 4, 300, 128, 32), (V2A, 3, 250, 256, 17), (V2, 2, 4000, 640, 30), (V2, 5, 4097, 128, 64), (V2, 6, 4200, 384, 33),
                                             (V2, 4, 4096, 14336, 8), (V2A, 2, 2500, 14336, 16), (V2, 3, 4096, 28672, 12)])
def test_resident_kernel(mode, bits, N, K, M):
    check(xi.random_weights(mode, bits, N, K, density=0.01 if K < 1024 else 0.002, seed=N + K), M, (RESIDENT, M))


@pytest.mark.parametrize("mode,bits,N,K,M", [(V2, 4, 1024, 512, 8), (V2, 4, 1024, 2048, 16), (V2, 2, 1024, 4096, 8), (V2A, 3, 1024, 4096, 16),
                                             (V2, 4, 4096, 14336, 8), (V2, 3, 4096, 28672, 12), (V2, 4, 2048, 20480, 16), (V2A, 4, 300, 256, 30),
                                             (V2A, 2, 600, 8192, 30), (V2, 4, 300, 8192, 64), (V2, 5, 8192, 4096, 8), (V2, 6, 8192, 1152, 16)])
def test_resident_sums_are_as_exact_as_token_by_token(mode, bits, N, K, M):
    """Against 64 bits, the fp32 results are no further off than those of the same tokens one by one, in the kernels with one chain
    per lane (5 % for what two samples of rounding errors differ by; measured 0.72 to 1.00)."""
    W = xi.random_weights(mode, bits, N, K, L=16, density=0.003, seed=K + bits)
    dW, x = xfp.upload(W), dev_x(xi.activations(np.random.default_rng(K), M, K))
    assert xfp.xfp_launch_route(dW, M) == (RESIDENT, M)
    dense = xfp.xfp_dequant_bulk(dW).view(torch.float16).double()
    ptr = torch.from_numpy(W.out_row_ptr.astype(np.int64)).cuda()
    rows = torch.repeat_interleave(torch.arange(N, device="cuda"), ptr[1:] - ptr[:-1])
    dense[rows, torch.from_numpy(W.out_col.astype(np.int64)).cuda()] += torch.from_numpy(W.out_val.view(np.float16).astype(np.float64)).cuda()
    exact = x.double() @ dense.T
    one_by_one = torch.cat([xfp.xfp_gemv(dW, x[m:m + 1], y_dtype=torch.float32) for m in range(M)])
    err = [float(((v.double() - exact).norm() / exact.norm()).item()) for v in (xfp.xfp_gemv(dW, x, y_dtype=torch.float32), one_by_one)]
    print(f"  {err[0]:.2e} {err[1]:.2e}", flush=True)
    assert err[0] <= 1.05 * err[1], err


@pytest.mark.parametrize("bits", [5, 6])
def test_resident_kernel_infinities_and_nan_stay_with_their_tokens(bits):
    W = xi.random_weights(V2, bits, 4100, 1152, density=0.01, seed=4)
    x, dW = dev_x(xi.activations(np.random.default_rng(5), 13, W.K)), xfp.upload(W)
    assert xfp.xfp_launch_route(dW, 13) == (RESIDENT, 13)
    clean = xfp.xfp_gemv(dW, x, y_dtype=torch.float32)
    x[3, 7], x[12, W.K - 1], x[0, 0] = float("inf"), float("nan"), float("-inf")
    y = xfp.xfp_gemv(dW, x, y_dtype=torch.float32)
    for m in range(13):
        if m == 12:
            assert torch.isnan(y[m]).all()
        elif m in (0, 3):                                             # (a codebook entry may be zero: no number there)
            assert not torch.isfinite(y[m]).any()
        else:
            assert torch.equal(y[m], clean[m])
