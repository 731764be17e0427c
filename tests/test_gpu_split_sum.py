"""Residual layers with their sum over K in parts (few tokens, a long K): through the block, which owns the scratch memory.
Against the oracle, and the same bits whether the layer runs whole or in panels behind streamed chunks, both streams of a
double-stream block in one launch or apart, one sample or several."""
import math

import numpy as np
import pytest
import torch

import workload as wl
from oracle import block as ob
from paper_2605_11335_amd import binding as B
from paper_2605_11335_amd.runner import BlockRunner
from tests.test_gpu_kernels import make_blob
from tests.util import bf16_round, dev_bits, max_abs, rel_l2

pytestmark = pytest.mark.gpu
BASE = dict(n_blocks=1, d=512, n_heads=4, head_dim=128, qk_rmsnorm=True, n_chunks=7)
CASES = {
    # K = 8768 and 137 slabs: no number of parts divides it
    "single": wl.BlockConfig("sum_single", wl.KIND_SINGLE, f=8256, n_total=301, **BASE),
    "dit": wl.BlockConfig("sum_dit", wl.KIND_DIT, f=8256, n_total=130, l_ctx=40, **BASE),
    "double": wl.BlockConfig("sum_double", wl.KIND_DOUBLE, f=8192, n_total=270, n_txt=70, **BASE),
}


def outputs(cfg, params, inputs, r):
    run = BlockRunner(cfg)
    try:
        run.ctx.set_resident_fraction(r)
        run.register_params(0, params)
        t = run.make_io(inputs)
        run.run_block(0, t)
        return {k: t[k].cpu().numpy() for k in ("y", "y_txt") if k in t}
    finally:
        run.close()


@pytest.mark.parametrize("name", sorted(CASES))
def test_sum_in_parts(name):
    cfg = CASES[name]
    params, inputs = wl.gen_block_params(cfg, 0), wl.gen_block_inputs(cfg, 0)
    got = outputs(cfg, params, inputs, 1.0)
    ref = ob.block_forward(cfg, params, inputs)
    for k, v in got.items():
        print(f"{name} {k}: rel_l2={rel_l2(v, ref[k]):.3e}", flush=True)
        assert rel_l2(v, ref[k]) <= 1e-2 and max_abs(v, ref[k]) <= 5e-2
    for r in (0.0, 0.6):
        for k, v in outputs(cfg, params, inputs, r).items():
            assert np.array_equal(v.view(np.uint8), got[k].view(np.uint8)), (r, k)
    both = cfg.with_(batch=2)
    two = outputs(both, params, wl.gen_block_inputs(both, 0), 1.0)
    for k, v in two.items():
        assert np.array_equal(np.ascontiguousarray(v[0]).view(np.uint8), got[k].view(np.uint8)), k


TILES = [(256, 256), (192, 256), (128, 256), (128, 128), (128, 64), (64, 64)]


@pytest.mark.parametrize("M,N,K,parts", [(700, 520, 1984, 3), (65, 264, 640, 2), (1, 8, 128, 2), (300, 1032, 2176, 5)])
def test_every_tile_and_both_ways_to_put_the_parts_together(M, N, K, parts):
    """The same bits from every tile, by the kernel that adds all parts and by the last part's own launch; right against float64.
    Ragged tokens, features and parts."""
    rng = np.random.default_rng(M + K)
    a, ab = bf16_round(rng.normal(size=(M, K)))
    buf, w, b, w_off, b_off = make_blob(rng, N, K)
    A, blob = dev_bits(ab), torch.from_numpy(buf).to("cuda:0")
    resid, gate = rng.normal(size=(M, N)).astype(np.float32), rng.normal(size=N).astype(np.float32)
    R, G = torch.from_numpy(resid).to("cuda:0"), torch.from_numpy(gate).to("cuda:0")
    ref = resid + gate.astype(np.float64) * (a.astype(np.float64) @ w.T + b)
    first = None
    for tile in TILES:
        for joins in (False, True):
            scratch = torch.full((parts * M * N,), float("nan"), device="cuda:0")
            y = torch.zeros((M, N), device="cuda:0")
            B.cf_op_linear_residual_form(A, blob, w_off, b_off, M, N, K, R, G, y, tile, parts, joins, scratch)
            torch.cuda.synchronize()
            # fp32 sums of K products of size 0.05: each rounding is at most 2^-24 of a partial sum of size 0.05 sqrt(K)
            assert max_abs(y.cpu().numpy(), ref) < 5e-5 * math.sqrt(K), (tile, joins)
            first = y if first is None else first
            assert torch.equal(y, first), (tile, joins)


@pytest.mark.parametrize("kind,n,txt,batch", [(wl.KIND_SINGLE, 700, 0, 8), (wl.KIND_DOUBLE, 647, 70, 6)])
def test_sum_in_parts_of_a_batch_that_fills_the_chip(kind, n, txt, batch):
    """There the last part's launch puts the sum together, of one layer and of the two streams'; every sample has the bits it has
    alone, where a kernel of its own does."""
    cfg = wl.BlockConfig("sum_batch", kind, n_blocks=1, d=1024, n_heads=8, head_dim=128, f=8192, n_total=n, n_txt=txt, qk_rmsnorm=True, n_chunks=5,
                         batch=batch)
    k = 1024 + 8192 if kind == wl.KIND_SINGLE else 8192
    alone, many = (B.cf_plan_block_linear(n - txt, 1024, k, True, rows2=txt, batch=b) for b in (1, batch))
    assert alone.parts == many.parts > 1 and not alone.last_tile_tokens and many.last_tile_tokens
    params = wl.gen_block_params(cfg, 0)
    got = outputs(cfg, params, wl.gen_block_inputs(cfg, 0), 1.0)
    one = cfg.with_(batch=1)
    for s in range(batch):
        for name, v in outputs(one, params, wl.gen_block_inputs(cfg, 0, sample=s), 1.0 if s else 0.0).items():
            assert np.array_equal(v.view(np.uint8), np.ascontiguousarray(got[name][s]).view(np.uint8)), (s, name)
