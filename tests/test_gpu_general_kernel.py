"""The general kernel's requests ahead of their use: odd and even numbers of steps of 64 units, rows of less than a step, several
rows of a wave and rows that are not there, more outliers than a wave's first request, every format that it takes."""
import numpy as np
import pytest
import torch

import oracle
import paper_2605_14844_amd as xfp
import xfp_inputs as xi
from helpers import gated_rel_err

pytestmark = pytest.mark.gpu
V2, V2A = xi.MODE_V2, xi.MODE_V2A


@pytest.mark.parametrize("mode,bits,N,K,L,affine,density", [
    (V2, 5, 1, 128, 0, False, 0.1), (V2, 6, 20011, 128, 0, False, 0.02), (V2, 5, 33001, 256, 0, False, 0.02), (V2, 6, 7, 2048, 0, False, 0.2), (V2, 5, 4099, 2176, 0, False, 0.005),
    (V2, 6, 301, 4224, 0, False, 0.03), (V2, 5, 130, 6144, 0, False, 0.01), (V2, 5, 66, 20480, 0, False, 0.01), (V2A, 5, 75, 4224, 16, False, 0.01),
    (V2A, 6, 41, 2176, 9, True, 0.01), (V2A, 3, 50, 18432, 32, True, 0.004), (V2A, 4, 37, 4224, 256, True, 0.01),
    # two and four rows of a wave, of two, three and four steps: the requests go on in the next row
    (V2, 5, 16399, 2176, 0, False, 0.004), (V2, 6, 16390, 4224, 0, False, 0.002), (V2, 5, 33001, 4352, 0, False, 0.0), (V2, 6, 16387, 6272, 0, False, 0.03)])
def test_general_kernel(mode, bits, N, K, L, affine, density):
    W = xi.random_weights(mode, bits, N, K, density=density, seed=N + K, **(dict(L=L, affine=affine) if mode == V2A else {}))
    x = xi.activations(np.random.default_rng(N + K), 1, K)
    dW, xd = xfp.upload(W), torch.from_numpy(x.view(np.int16)).cuda().view(torch.float16)
    assert xfp.xfp_launch_route(dW, 1) == (xfp.XFP_ROUTE_GENERAL, 1)
    y = xfp.xfp_gemv(dW, xd, y_dtype=torch.float32)
    torch.cuda.synchronize()
    assert gated_rel_err(y.cpu().numpy().astype(np.float64), oracle.gemv_weights(W, x)) <= 1e-4      # fp32 results, as in the other kernels' tests
    xb = xd.float().bfloat16()                                        # bf16 activations: the converted call's bits
    assert torch.equal(xfp.xfp_gemv(dW, xb, y_dtype=torch.float32), xfp.xfp_gemv(dW, xfp.xfp_convert_bf16_to_f16(xb), y_dtype=torch.float32))
