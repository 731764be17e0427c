"""The tile shapes of the linear layers (256x256, 192x256, 128x256, 128x128, 128x64, 64x64 tokens x features): which one a launch
takes depends on its size, the order of every sum does not, so the rows of a large launch equal, bit for bit, the same rows
computed by launches of fewer tokens; and the large launch is right against the float64 product.  Every epilogue (either
activation, the gated residual) on every tile, and on every tile two layers in one launch."""
import math

import numpy as np
import pytest
import torch

import workload as wl
from oracle import block as ob
from paper_2605_11335_amd import binding as B
from paper_2605_11335_amd.runner import BlockRunner
from tests.test_gpu_kernels import make_blob
from tests.util import assert_bf16_close, bf16_round, dev_bits, host_bits, max_abs, rel_l2

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
M, N = 2500, 4616                                # ragged for every tile
FEWER = (1, 63, 65, 200, 370, 500, 1100, 1290, 1900, 2250)
KS = (64, 128, 192, 448, 832)                    # slabs of 64: fewer than a ring has stages, odd and even counts, more than any ring holds
TILES = {(256, 256), (192, 256), (128, 256), (128, 128), (128, 64), (64, 64)}


@pytest.mark.parametrize("K", KS)
def test_every_tile_shape_gives_the_same_bits(K):
    rng = np.random.default_rng(K)
    a, ab = bf16_round(rng.normal(size=(M, K)))
    buf, w, b, w_off, b_off = make_blob(rng, N, K)
    A, blob = dev_bits(ab), torch.from_numpy(buf).to(DEV)
    resid = torch.from_numpy(rng.normal(size=(M, N)).astype(np.float32)).to(DEV)
    gate = torch.from_numpy(rng.normal(size=N).astype(np.float32)).to(DEV)

    def layer(m):
        out = torch.zeros((m, N), dtype=torch.int16, device=DEV)
        erf = torch.zeros_like(out)
        y = torch.zeros((m, N), dtype=torch.float32, device=DEV)
        B.cf_op_linear(A, blob, w_off, b_off, m, N, K, None, out, n_split=0)
        B.cf_op_linear(A, blob, w_off, b_off, m, N, K, None, erf, n_split=0, gelu_erf=True)
        B.cf_op_linear_residual(A, blob, w_off, b_off, m, N, K, resid, gate, y)
        torch.cuda.synchronize()
        return out, y, erf

    out, y, erf = layer(M)
    z = a.astype(np.float64) @ w.T + b
    assert_bf16_close(host_bits(out), ob.gelu_tanh(z), extra_abs=2e-4)
    assert_bf16_close(host_bits(erf), ob.gelu_erf(z), extra_abs=2e-4)
    # fp32 sums of K products of size 0.05: each rounding is at most 2^-24 of a partial sum of size 0.05 sqrt(K)
    assert max_abs(y.cpu().numpy(), resid.cpu().numpy().astype(np.float64) + gate.cpu().numpy().astype(np.float64) * z) < 5e-5 * math.sqrt(K)
    for m in FEWER:
        o, v, e = layer(m)
        assert torch.equal(o, out[:m]) and torch.equal(v, y[:m]) and torch.equal(e, erf[:m]), m
    # the same features as panels of a few tiles each
    o = torch.zeros_like(out)
    for n0, n1 in ((0, 64), (64, 584), (584, 2048), (2048, N)):
        B.cf_op_linear(A, blob, w_off, b_off, M, N, K, None, o, n_split=0, n0=n0, n1=n1)
    torch.cuda.synchronize()
    assert torch.equal(o, out)


TXT = 70
IMAGES = (300, 700, 1000, 4000, 6000, 8000)


@pytest.mark.parametrize("erf", [False, True])
@pytest.mark.parametrize("img", IMAGES)
def test_two_streams_in_one_launch(img, erf):
    """The MLP-in layer of a double-stream block takes each of the tiles above for both streams at once when its weights are in
    place, and launches of their own per stream and panel when they are streamed: the same bits, and right against the oracle."""
    cfg = wl.BlockConfig("pair", wl.KIND_DOUBLE, n_blocks=1, d=512, n_heads=4, head_dim=128, f=2048, n_total=img + TXT, n_txt=TXT, qk_rmsnorm=True,
                         n_chunks=9, gelu_erf=erf)
    params, inputs = wl.gen_block_params(cfg, 0), wl.gen_block_inputs(cfg, 0)
    got = []
    for r in (1.0, 0.0):
        run = BlockRunner(cfg)
        try:
            run.ctx.set_resident_fraction(r)
            run.register_params(0, params)
            t = run.make_io(inputs)
            run.run_block(0, t)
            got.append(np.concatenate([t["y_txt"].cpu().numpy(), t["y"].cpu().numpy()]))
        finally:
            run.close()
    assert np.array_equal(got[0].view(np.uint8), got[1].view(np.uint8))
    rows = np.sort(np.random.default_rng(img).choice(img + TXT, 150, replace=False))
    ref = ob.block_forward(cfg, params, inputs, rows=rows)["y_rows"]
    assert rel_l2(got[0][rows], ref) <= 1e-2
