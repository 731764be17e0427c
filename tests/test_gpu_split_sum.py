"""Residual layers with their sum over K in parts (few tokens, a long K): through the block, which owns the scratch memory.
Against the oracle, and the same bits whether the layer runs whole or in panels behind streamed chunks, both streams of a
double-stream block in one launch or apart, one sample or several."""
import numpy as np
import pytest

import workload as wl
from oracle import block as ob
from paper_2605_11335_amd.runner import BlockRunner
from tests.util import max_abs, rel_l2

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
