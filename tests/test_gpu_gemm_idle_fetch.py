"""Launches whose last round of workgroups leaves CUs idle, on the three largest tiles (one workgroup per CU): from 16 slabs on,
workgroups without a tile fetch operands ahead there.  One tile and all but one of a round, ragged rows, features and slabs, a sum in
parts; and the two streams of a double-stream block in one launch, with the weights in one buffer and split between two."""
import math

import numpy as np
import pytest
import torch

import workload as wl
from paper_2605_11335_amd import binding as B
from paper_2605_11335_amd.runner import BlockRunner
from tests.test_gpu_kernels import make_blob
from tests.util import bf16_round, dev_bits, max_abs

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("tile", [(256, 256), (192, 256), (128, 256)])
@pytest.mark.parametrize("M,N,K,parts", [(5, 8, 1024, 1), (300, 520, 1088, 1), (1500, 3080, 1984, 1), (700, 1032, 3968, 2), (3300, 5000, 1152, 1)])
def test_last_round(tile, M, N, K, parts):
    rng = np.random.default_rng(M + K)
    a, ab = bf16_round(rng.normal(size=(M, K)))
    buf, w, b, w_off, b_off = make_blob(rng, N, K)
    resid = torch.from_numpy(rng.normal(size=(M, N)).astype(np.float32)).to(DEV)
    gate = torch.from_numpy(rng.normal(size=N).astype(np.float32)).to(DEV)
    y = torch.full((M, N), float("nan"), dtype=torch.float32, device=DEV)
    scratch = torch.empty(parts * M * N, dtype=torch.float32, device=DEV) if parts > 1 else None
    B.cf_op_linear_residual_form(dev_bits(ab), torch.from_numpy(buf).to(DEV), w_off, b_off, M, N, K, resid, gate, y, tile, parts, False, scratch)
    torch.cuda.synchronize()
    ref = resid.cpu().numpy().astype(np.float64) + gate.cpu().numpy().astype(np.float64) * (a.astype(np.float64) @ w.T + b)
    # fp32 sums of K products of size 0.05: each rounding is at most 2^-24 of a partial sum of size 0.05 sqrt(K)
    assert max_abs(y.cpu().numpy(), ref) < 5e-5 * math.sqrt(K)


@pytest.mark.parametrize("img", [300, 1500])
def test_two_streams(img):
    cfg = wl.BlockConfig("idle_pair", wl.KIND_DOUBLE, n_blocks=1, d=1024, n_heads=8, head_dim=128, f=4096, n_total=img + 70, n_txt=70, qk_rmsnorm=True, n_chunks=9)
    params, inputs = wl.gen_block_params(cfg, 0), wl.gen_block_inputs(cfg, 0)
    got = []
    for r in (1.0, 0.5, 0.0):
        run = BlockRunner(cfg)
        try:
            run.ctx.set_resident_fraction(r)
            run.register_params(0, params)
            t = run.make_io(inputs)
            run.run_block(0, t)
            got.append(np.concatenate([t["y_txt"].cpu().numpy(), t["y"].cpu().numpy()]))
        finally:
            run.close()
    assert np.isfinite(got[0]).all()
    for g in got[1:]:
        assert np.array_equal(g.view(np.uint8), got[0].view(np.uint8))
