"""Residual layers with their sum over K in two or three parts whose workgroups put it together within the launch: one layer on every tile, and in
the blocks that launch it so, of one sample and of several, one layer and the two of a double-stream block."""
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
TILES = [(256, 256), (192, 256), (128, 256), (128, 128), (128, 64), (64, 64)]


# ragged tokens, features and parts; one output row; more workgroups of every tile than run at once (4100 x 1800: 272 of the largest in two
# parts, 3900 x 1800: 384 in three), so that some parts find the others not begun and one of them finishes the tile
@pytest.mark.parametrize("M,N,K,parts", [(700, 520, 1984, 3), (65, 264, 640, 2), (1, 8, 128, 2), (300, 1032, 2176, 2), (3900, 1800, 256, 2), (3900, 1800, 320, 3), (4100, 1800, 256, 2)])
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


SINGLE, DIT, DOUBLE = wl.KIND_SINGLE, wl.KIND_DIT, wl.KIND_DOUBLE
# kind, d, f, tokens (text tokens of them), batch; the tile and the parts that the last layer meets on
BLOCKS = [(SINGLE, 512, 4096, 856, 0, 4, (128, 128), 2), (SINGLE, 1024, 4096, 616, 0, 4, (128, 256), 3), (SINGLE, 1024, 4096, 1168, 0, 3, (192, 256), 3),
          (SINGLE, 1024, 4096, 1168, 0, 4, (256, 256), 3), (DIT, 1536, 6144, 880, 0, 3, (192, 256), 3), (DOUBLE, 1024, 6144, 1312, 72, 1, (128, 128), 2),
          (DOUBLE, 1024, 4096, 352, 72, 4, (128, 128), 2), (DOUBLE, 1024, 6144, 616, 40, 4, (128, 256), 3), (DOUBLE, 1024, 6144, 1312, 72, 2, (128, 256), 2),
          (DOUBLE, 1024, 6144, 1312, 72, 4, (192, 256), 2), (DOUBLE, 1024, 8192, 664, 40, 4, (192, 256), 3)]


def forwards(cfg, params, resident, *inputs):
    """Outputs of one forward after the other, all on one workspace."""
    run = BlockRunner(cfg)
    try:
        run.ctx.set_resident_fraction(resident)
        run.register_params(0, params)
        out = []
        for i in inputs:
            t = run.make_io(i)
            run.run_block(0, t)
            out.append({k: t[k].cpu().numpy() for k in ("y", "y_txt") if k in t})
        return out
    finally:
        run.close()


@pytest.mark.parametrize("kind,d,f,n,txt,batch,tile,parts", BLOCKS)
def test_blocks_whose_parts_meet(kind, d, f, n, txt, batch, tile, parts):
    """Every sample of a batch has the bits it has alone, where a kernel adds the parts on other tiles, or while weights stream, in panels; a forward
    has the same bits before and after another one, which leaves its words and sums in the workspace; and they are right against the oracle."""
    k = d + f if kind == SINGLE else f
    p = B.cf_plan_block_linear(n - txt, d, k, True, rows2=txt, batch=batch)
    assert ((p.tile_tokens, p.tile_features), p.parts) == (tile, parts) and B.cf_plan_block_meet(n - txt, d, k, rows2=txt, batch=batch)
    cfg = wl.BlockConfig("sum_meets", kind, n_blocks=1, d=d, n_heads=d // 128, head_dim=128, f=f, n_total=n, n_txt=txt, l_ctx=40 if kind == DIT else 0, qk_rmsnorm=True,
                         n_chunks=5, batch=batch)
    print(cfg, flush=True)
    params, inputs = wl.gen_block_params(cfg, 0), wl.gen_block_inputs(cfg, 0)
    got, _, again = forwards(cfg, params, 1.0, inputs, wl.gen_block_inputs(cfg, 1), inputs)
    for key in got:
        assert np.isfinite(got[key]).all() and np.array_equal(got[key].view(np.uint8), again[key].view(np.uint8)), key
    one = cfg.with_(batch=1)
    for s in range(batch):
        i = wl.gen_block_inputs(cfg, 0, sample=s) if batch > 1 else inputs
        for key, v in forwards(one, params, float(s % 2), i)[0].items():
            assert np.array_equal(v.view(np.uint8), np.ascontiguousarray(got[key][s] if batch > 1 else got[key]).view(np.uint8)), (s, key)
        if s == batch - 1:
            rows = np.sort(np.random.default_rng(n).choice(n, 40, replace=False))
            ref = ob.block_forward(one, params, i, rows=rows)["y_rows" if kind == DOUBLE else "y"]
            y = [got[key][s] if batch > 1 else got[key] for key in (("y_txt", "y") if kind == DOUBLE else ("y",))]
            assert rel_l2(np.concatenate(y)[rows], ref) <= 1e-2
