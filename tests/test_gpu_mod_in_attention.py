"""Modulation vectors that only what follows attention needs (gates, the MLP's shift and scale), computed by workgroups behind those of
attention: against the oracle, and the same bits as where the weights still stream and every vector is computed ahead."""
import numpy as np
import pytest

import workload as wl
from oracle import block as ob
from paper_2605_11335_amd import binding as B
from paper_2605_11335_amd.runner import BlockRunner
from tests.util import max_abs, rel_l2

pytestmark = pytest.mark.gpu
BASE = dict(n_blocks=1, qk_rmsnorm=True, n_chunks=9)
# sweeps as one workgroup (4 or 8 waves), in parts with a merge kernel, 64-wide heads, a batch whose parts are in one workgroup; K of three and four steps
CASES = {
    "single": wl.BlockConfig("mod_single", wl.KIND_SINGLE, d=1536, n_heads=12, head_dim=128, f=512, n_total=2100, **BASE),
    "single64": wl.BlockConfig("mod_single64", wl.KIND_SINGLE, d=512, n_heads=8, head_dim=64, f=512, n_total=2600, **BASE),
    "dit": wl.BlockConfig("mod_dit", wl.KIND_DIT, d=1024, n_heads=8, head_dim=128, f=512, n_total=1800, l_ctx=40, **BASE),
    "double": wl.BlockConfig("mod_double", wl.KIND_DOUBLE, d=1536, n_heads=12, head_dim=128, f=512, n_total=2000, n_txt=80, sp_degree=2, sp_rank=1, **BASE),
    "double_batch": wl.BlockConfig("mod_double_batch", wl.KIND_DOUBLE, d=512, n_heads=4, head_dim=128, f=512, n_total=1500, n_txt=70, batch=2, **BASE),
}


def outputs(cfg, params, inputs, r):
    """-> operations of the product launched ahead of the block, outputs"""
    run = BlockRunner(cfg)
    try:
        run.ctx.set_resident_fraction(r)
        run.register_params(0, params)
        t = run.make_io(inputs)
        run.ctx.cf_set_profiling(True)
        run.run_block(0, t)
        run.ctx.cf_sync()
        ahead = sum(k["flops"] for k in run.ctx.cf_kernel_times() if k["name"] == "modvec")
        return ahead, {k: t[k].cpu().numpy() for k in ("y", "y_txt") if k in t}
    finally:
        run.close()


@pytest.mark.parametrize("name", sorted(CASES))
def test_vectors_computed_beside_attention(name):
    cfg = CASES[name]
    heads, batch = cfg.n_heads // cfg.sp_degree, max(1, cfg.batch)
    p = B.cf_plan_block_attention(heads, batch, cfg.n_total, cfg.n_total, cfg.head_dim)
    groups = -(-cfg.n_total // (32 * p.waves)) * heads * batch * (1 if p.all_parts else p.parts)
    print(name, p.parts, p.all_parts, p.deal, p.waves, groups, flush=True)
    assert p.deal == 0 and p.all_parts != 2 and groups <= 224 * (2 if p.waves == 4 else 1) * (2 if cfg.head_dim == 64 else 1)
    params, inputs = wl.gen_block_params(cfg, 0), wl.gen_block_inputs(cfg, 0)
    ahead, got = outputs(cfg, params, inputs, 1.0)
    whole, streamed = outputs(cfg, params, inputs, 0.0)
    # two of three vectors (of six, of each stream's six) go ahead, the others beside attention; while weights stream all of them
    vectors = {wl.KIND_SINGLE: 3, wl.KIND_DIT: 6, wl.KIND_DOUBLE: 12}[cfg.kind]
    first = 4 if cfg.kind == wl.KIND_DOUBLE else 2
    assert (ahead, whole) == tuple(2.0 * batch * v * cfg.d * cfg.d for v in (first, vectors))
    for k, v in streamed.items():
        assert np.array_equal(v.view(np.uint8), got[k].view(np.uint8)), k
    if batch == 1:
        ref = ob.block_forward(cfg, params, inputs)
        for k, v in got.items():
            assert rel_l2(v, ref[k]) <= 1e-2 and max_abs(v, ref[k]) <= 5e-2, k
