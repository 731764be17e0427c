"""Attention dealt out by the kernel (a sweep that one workgroup begins and another ends), in even shares and as the workgroups
come for it: against the oracle, and the same bits as sweeps done by one workgroup each -- a batch large enough to be dealt out
equals its samples run alone, which are too small for it (or, the long ones, are dealt out differently).  Sweeps that have to be
repeated are compared bit for bit in test_gpu_attention_forms.py."""
import numpy as np
import pytest

import workload as wl
from oracle import block as ob
from paper_2605_11335_amd.runner import BlockRunner
from tests.util import rel_l2

pytestmark = pytest.mark.gpu


def forward(cfg, params, inputs):
    run = BlockRunner(cfg)
    try:
        run.ctx.set_resident_fraction(1.0)
        run.register_params(0, params)
        t = run.make_io(inputs)
        run.run_block(0, t)
        return t["y"].cpu().numpy()
    finally:
        run.close()


# query tiles of 256: 12 x 24 heads = 9 groups of 32 exactly; 11 x 24 (one sample, or two of 12 heads) = 8 groups and a quarter.
# 353 x 6 = 66 groups and 6 tiles, of sweeps long enough to be drawn from a counter
@pytest.mark.parametrize("n,heads,hd,batch,sharp", [(2850, 24, 128, 1, 1.0), (2760, 24, 128, 1, 1.0), (2760, 12, 128, 2, 1.0), (2760, 24, 128, 1, 20.0),
                                                     (90200, 2, 128, 3, 1.0)])
def test_dealt_out_evenly(n, heads, hd, batch, sharp):
    cfg = wl.BlockConfig("even", wl.KIND_SINGLE, n_blocks=1, d=heads * hd, n_heads=heads, head_dim=hd, f=256, n_total=n, n_chunks=3, batch=batch)
    params, inputs = wl.gen_block_params(cfg, 0), wl.gen_block_inputs(cfg, 0)
    for k in ("q_norm", "k_norm"):
        params[k] = wl.f32_to_bf16_bits(wl.bf16_bits_to_f32(params[k]) * np.float32(np.sqrt(sharp)))
    y = forward(cfg, params, inputs).reshape(batch, n, -1)
    one = cfg.with_(batch=1)
    for b in range(batch):
        x = wl.gen_block_inputs(cfg, 0, sample=b)
        if batch > 1:
            assert np.array_equal(forward(one, params, x).view(np.uint8), np.ascontiguousarray(y[b]).view(np.uint8)), b
        rows = np.sort(np.random.default_rng(b).choice(n, 200, replace=False))
        ref = ob.block_forward(one, params, x, rows=rows)["y"]
        print(f"sample {b}: rel_l2={rel_l2(y[b][rows], ref):.3e}", flush=True)
        # a logit of standard deviation 20 moves by 0.05 when q and k are rounded to bf16, and its weight by as many per cent;
        # tiles then go out of the fast softmax's range, and the sweep is repeated by the workgroup with its last piece
        assert rel_l2(y[b][rows], ref) <= (1e-2 if sharp == 1.0 else 5e-2)
