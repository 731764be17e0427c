"""The tile shapes of the linear layers (256x256, 192x256, 128x256, 128x128, 128x64, 64x64 tokens x features): which one a launch
takes depends on its size, the order of every sum does not, so the rows of a large launch equal, bit for bit, the same rows
computed by launches of fewer tokens; and the large launch is right against the float64 product."""
import math

import numpy as np
import pytest
import torch

from oracle import block as ob
from paper_2605_11335_amd import binding as B
from tests.test_gpu_kernels import make_blob
from tests.util import assert_bf16_close, bf16_round, dev_bits, host_bits, max_abs

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
M, N = 2500, 4616                                # ragged for every tile


# slabs of 64: fewer than a ring has stages, odd and even counts, more than any ring holds
@pytest.mark.parametrize("K", [64, 128, 192, 448, 832])
def test_every_tile_shape_gives_the_same_bits(K):
    rng = np.random.default_rng(K)
    a, ab = bf16_round(rng.normal(size=(M, K)))
    buf, w, b, w_off, b_off = make_blob(rng, N, K)
    A, blob = dev_bits(ab), torch.from_numpy(buf).to(DEV)
    resid = torch.from_numpy(rng.normal(size=(M, N)).astype(np.float32)).to(DEV)
    gate = torch.from_numpy(rng.normal(size=N).astype(np.float32)).to(DEV)

    def layer(m):
        out = torch.zeros((m, N), dtype=torch.int16, device=DEV)
        y = torch.zeros((m, N), dtype=torch.float32, device=DEV)
        B.cf_op_linear(A, blob, w_off, b_off, m, N, K, None, out, n_split=0)
        B.cf_op_linear_residual(A, blob, w_off, b_off, m, N, K, resid, gate, y)
        torch.cuda.synchronize()
        return out, y

    out, y = layer(M)
    z = a.astype(np.float64) @ w.T + b
    assert_bf16_close(host_bits(out), ob.gelu_tanh(z), extra_abs=2e-4)
    # fp32 sums of K products of size 0.05: each rounding is at most 2^-24 of a partial sum of size 0.05 sqrt(K)
    assert max_abs(y.cpu().numpy(), resid.cpu().numpy().astype(np.float64) + gate.cpu().numpy().astype(np.float64) * z) < 5e-5 * math.sqrt(K)
    for m in (1, 63, 65, 200, 500, 1100, 1900, 2250):
        o, v = layer(m)
        assert torch.equal(o, out[:m]) and torch.equal(v, y[:m]), m
    # the same features as panels of a few tiles each
    o = torch.zeros_like(out)
    for n0, n1 in ((0, 64), (64, 584), (584, 2048), (2048, N)):
        B.cf_op_linear(A, blob, w_off, b_off, M, N, K, None, o, n_split=0, n0=n0, n1=n1)
    torch.cuda.synchronize()
    assert torch.equal(o, out)
