"""Projections that place their heads themselves (normed, rotated, own v turned round, other heads to the send buffers) instead of
leaving rows for a pass of their own: on every tile, with heads of either width, at sizes where slices of 32 tokens straddle samples, segments
and the ends of the problem.  With all weights in place the launch places them where that is estimated to pay; while weights
stream, their panels leave rows for the pass.  The arithmetic is the same, so all outputs are, bit for bit; and they are right against the
oracle."""
import numpy as np
import pytest

import workload as wl
from oracle import block as ob
from paper_2605_11335_amd.runner import BlockRunner
from tests.util import rel_l2

pytestmark = pytest.mark.gpu
SINGLE, DIT, DOUBLE = wl.KIND_SINGLE, wl.KIND_DIT, wl.KIND_DOUBLE


def outputs(cfg, params, inputs, r):
    """-> launches of the pass over rows, bytes they move (none of rows that are placed), tiles of the q, k, v projection, outputs"""
    run = BlockRunner(cfg)
    try:
        run.ctx.set_resident_fraction(r)
        run.register_params(0, params)
        t = run.make_io(inputs)
        run.ctx.cf_set_profiling(True)
        run.run_block(0, t)
        run.ctx.cf_sync()
        times = [k for k in run.ctx.cf_kernel_times() if k["launches"]]
        passes, moved = (sum(k[what] for k in times if k["name"] == "pre_attention") for what in ("launches", "bytes"))
        tiles = [k["name"].split("/")[1] for k in times if k["name"].startswith(("gemm_lin1/", "gemm_qkv/"))]
        return passes, moved, tiles, {k: v.cpu().numpy().copy() for k, v in t.items() if k in ("y", "y_txt", "send_q", "send_k", "send_v", "send_attn")}
    finally:
        run.close()


def block(kind, d, hd, n, txt=0, sp=1, rank=0, batch=1, norm=True, rope=False, erf=False):
    return wl.BlockConfig(f"heads_{kind}_{d}_{n}", kind, n_blocks=1, d=d, n_heads=d // hd, head_dim=hd, f=2 * d, n_total=n, sp_degree=sp, sp_rank=rank, n_txt=txt,
                          l_ctx=77 if kind == DIT else 0, qk_rmsnorm=norm, rope=rope, gelu_erf=erf, batch=batch, n_chunks=12)


# kind, d, head width, tokens (text tokens of them), Ulysses degree and rank, batch, norm, tables, erf
CASES = [(SINGLE, 512, 64, 512, 0, 1, 0, 1, False, False, False), (SINGLE, 512, 64, 333, 0, 1, 0, 1, True, False, False), (SINGLE, 512, 64, 72, 0, 1, 0, 5, True, True, False),
         (SINGLE, 512, 128, 296, 0, 1, 0, 2, False, True, True), (SINGLE, 512, 128, 2000, 0, 2, 1, 1, True, False, False), (SINGLE, 1024, 128, 4624, 0, 2, 1, 1, True, False, False),
         (SINGLE, 1024, 64, 2328, 0, 1, 0, 2, True, True, False), (SINGLE, 1536, 128, 5001, 0, 1, 0, 1, True, False, True), (SINGLE, 2048, 128, 2640, 0, 2, 1, 1, True, False, False),
         (SINGLE, 512, 64, 5, 0, 1, 0, 40, True, False, False), (SINGLE, 512, 64, 333, 0, 1, 0, 3, False, False, False), (SINGLE, 512, 64, 5, 0, 1, 0, 1, False, False, False),
         (DIT, 512, 64, 592, 0, 2, 1, 1, True, False, False), (DIT, 512, 128, 592, 0, 2, 0, 2, False, False, True), (DIT, 1536, 128, 1320, 0, 1, 0, 1, True, False, False),
         (DOUBLE, 512, 64, 672, 64, 2, 1, 1, False, False, False), (DOUBLE, 1024, 128, 3050, 72, 1, 0, 1, True, True, False), (DOUBLE, 1024, 128, 912, 144, 1, 0, 3, True, False, True)]


@pytest.mark.parametrize("kind,d,hd,n,txt,sp,rank,batch,norm,rope,erf", CASES)
def test_placed_heads_are_those_of_the_pass(kind, d, hd, n, txt, sp, rank, batch, norm, rope, erf):
    cfg = block(kind, d, hd, n, txt, sp, rank, batch, norm, rope, erf)
    params, inputs = wl.gen_block_params(cfg, 0), wl.gen_block_inputs(cfg, 0)
    print(cfg, flush=True)
    passes, _, _, placed = outputs(cfg, params, inputs, 1.0)
    passes_streamed, _, _, rows = outputs(cfg, params, inputs, 0.0)
    assert passes <= passes_streamed
    if sp == 1:                                    # whether the launch is gone: only where v goes out eight tokens at a time
        assert (passes < passes_streamed) == (batch == 1 or (n % 8 == 0 and n >= 64)), (passes, passes_streamed)
    assert set(placed) == set(rows)
    for k in placed:
        assert np.isfinite(placed[k].astype(np.float32) if placed[k].dtype != np.int16 else 0).all()
        assert np.array_equal(placed[k].view(np.uint8), rows[k].view(np.uint8)), k
    if batch == 1:
        sample = np.sort(np.random.default_rng(n).choice(cfg.n_local, min(cfg.n_local, 60), replace=False))
        ref = ob.block_forward(cfg, params, inputs, rows=sample)["y_rows" if kind == DOUBLE else "y"]
        got = np.concatenate([placed["y_txt"], placed["y"]]) if kind == DOUBLE else placed["y"]
        assert rel_l2(got[sample], ref) <= 1e-2


@pytest.mark.parametrize("kind,d,hd,n,txt", [(DOUBLE, 1024, 128, 1280, 64), (DOUBLE, 1536, 64, 816, 272), (SINGLE, 512, 64, 352, 0), (SINGLE, 512, 64, 176, 0)])
def test_few_rows_beside_the_peers_go_through_the_pass(kind, d, hd, n, txt):
    """Whose launch is there in any case: on small tiles placing them costs more than their share of it."""
    cfg = block(kind, d, hd, n, txt, sp=2, rank=1, rope=kind == DOUBLE)
    params, inputs = wl.gen_block_params(cfg, 0), wl.gen_block_inputs(cfg, 0)
    _, moved, tiles, _ = outputs(cfg, params, inputs, 1.0)
    _, moved_streamed, _, _ = outputs(cfg, params, inputs, 0.0)
    print(cfg, tiles, moved, flush=True)
    assert tiles in (["64x64"], ["128x64"], ["128x128"]) and moved == moved_streamed > 0


# ranks' shares, with own and other heads side by side in a tile: staged whole by the waves of the same tokens, or (256 features) quadrant by quadrant
@pytest.mark.parametrize("kind,d,hd,n,txt,rank,norm,rope,tile",
                         [(DOUBLE, 512, 64, 2080, 80, 1, True, False, "64x64"), (DOUBLE, 512, 64, 2288, 80, 1, False, False, "128x64"), (DOUBLE, 1024, 128, 3488, 80, 1, True, True, "128x128"),
                          (DOUBLE, 1024, 64, 4080, 80, 0, True, False, "128x256"), (SINGLE, 1536, 128, 5008, 0, 1, True, False, "192x256"), (SINGLE, 1024, 128, 9248, 0, 1, True, True, "192x256"),
                          (SINGLE, 2048, 128, 9248, 0, 0, True, True, "256x256"), (SINGLE, 2048, 128, 9248, 0, 1, True, False, "256x256"),
                          (DOUBLE, 1024, 64, 8064, 80, 1, True, False, "256x256")])
def test_ranks_place_their_heads_on_every_tile(kind, d, hd, n, txt, rank, norm, rope, tile):
    cfg = block(kind, d, hd, n, txt, 2, rank, 1, norm, rope)
    params, inputs = wl.gen_block_params(cfg, 0), wl.gen_block_inputs(cfg, 0)
    _, moved, tiles, placed = outputs(cfg, params, inputs, 1.0)
    _, moved_rows, _, rows = outputs(cfg, params, inputs, 0.0)
    print(cfg, tiles, moved, moved_rows, flush=True)
    assert tiles == [tile] and moved == moved_rows - 4.0 * cfg.n_local * 3 * d        # the rows' part of the pass
    for k in placed:
        assert np.array_equal(placed[k].view(np.uint8), rows[k].view(np.uint8)), k
