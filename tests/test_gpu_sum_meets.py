"""Residual layers with their sum over K in two or three parts whose workgroups put it together within the launch."""
import math

import numpy as np
import pytest
import torch

from paper_2605_11335_amd import binding as B
from tests.test_gpu_kernels import make_blob
from tests.util import bf16_round, dev_bits, max_abs

pytestmark = pytest.mark.gpu
TILES = [(256, 256), (192, 256), (128, 256), (128, 128), (128, 64), (64, 64)]


# ragged tokens, features and parts; one output row; more workgroups of every tile than run at once (3900 x 1800: 256 of the largest in two
# parts), so that some parts find the others not begun and one of them finishes the tile
@pytest.mark.parametrize("M,N,K,parts", [(700, 520, 1984, 3), (65, 264, 640, 2), (1, 8, 128, 2), (300, 1032, 2176, 2), (3900, 1800, 256, 2), (3900, 1800, 320, 3)])
def test_parts_that_meet_give_the_bits_of_the_kernel_that_adds_them(M, N, K, parts):
    rng = np.random.default_rng(M + K)
    a, ab = bf16_round(rng.normal(size=(M, K)))
    buf, w, b, w_off, b_off = make_blob(rng, N, K)
    A, blob = dev_bits(ab), torch.from_numpy(buf).to("cuda:0")
    resid, gate = rng.normal(size=(M, N)).astype(np.float32), rng.normal(size=N).astype(np.float32)
    R, G = torch.from_numpy(resid).to("cuda:0"), torch.from_numpy(gate).to("cuda:0")
    ref = resid + gate.astype(np.float64) * (a.astype(np.float64) @ w.T + b)
    added = torch.zeros((M, N), device="cuda:0")
    B.cf_op_linear_residual_form(A, blob, w_off, b_off, M, N, K, R, G, added, (128, 128), parts, False, torch.empty(parts * M * N, device="cuda:0"))
    # fp32 sums of K products of size 0.05: each rounding is at most 2^-24 of a partial sum of size 0.05 sqrt(K)
    assert max_abs(added.cpu().numpy(), ref) < 5e-5 * math.sqrt(K)
    for tile in TILES:
        tiles = -(-M // tile[0]) * -(-N // tile[1])
        for gate_here in (G, None):
            scratch = torch.full((4 * tiles + parts * tiles * tile[0] * tile[1],), float("nan"), device="cuda:0")
            scratch[:4 * tiles] = 0
            y = torch.full((M, N), float("nan"), device="cuda:0")
            print(tile, gate_here is None, flush=True)
            B.cf_op_linear_residual_form(A, blob, w_off, b_off, M, N, K, R, gate_here, y, tile, parts, 2, scratch)
            torch.cuda.synchronize()
            if gate_here is not None:
                assert torch.equal(y, added), tile
            else:
                assert max_abs(y.cpu().numpy(), resid + (ref - resid) / gate) < 5e-5 * math.sqrt(K), tile


def test_words_and_parts_are_checked():
    t = torch.zeros(1 << 16, device="cuda:0")
    for parts, floats in ((2, 4 + 2 * 64 * 64 - 1), (4, 1 << 16)):
        with pytest.raises(B.ChunkflowError):
            B.cf_op_linear_residual_form(t, t, 0, 1 << 15, 64, 64, 256, t, None, t, (64, 64), parts, 2, t[:floats])
