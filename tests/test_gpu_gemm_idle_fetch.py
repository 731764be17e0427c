"""Launches whose last round of workgroups leaves CUs idle, on the three largest tiles (one workgroup per CU): from 16 slabs on and up to
two rounds, workgroups without a tile fetch operands ahead there (what they read is checked on the host, test_abi.py).  One tile and all but one of a round, ragged rows, features and slabs, a sum in
parts; and the two streams of a double-stream block in one launch, with the weights in one buffer and split between two."""
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
DEV = "cuda:0"


@pytest.mark.parametrize("tile", [(256, 256), (192, 256), (128, 256)])
@pytest.mark.parametrize("M,N,K,parts", [(5, 8, 1024, 1), (300, 520, 1088, 1), (1500, 3080, 1984, 1), (700, 1032, 3968, 2), (3300, 5000, 1152, 1), (3300, 4608, 1152, 1)])
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


def paired_layers(cfg):
    """(name, tile, whether idle CUs fetch) of a double-stream block's paired layers, from the planner."""
    d, f, img, txt = cfg.d, cfg.f, cfg.n_total - cfg.n_txt, cfg.n_txt
    for name, n, k, residual in (("qkv", 3 * d, d, False), ("out", d, d, True), ("up", f, d, False), ("down", d, f, True)):
        p = B.cf_plan_block_linear(img, n, k, residual, rows2=txt)
        yield name, f"{p.tile_tokens}x{p.tile_features}", p.parts, B.cf_plan_block_fetch(img, n, k, residual, rows2=txt).fetching > 0


# between them every paired kernel that can fetch: both tiles, plain, either activation, residual, parts of a cut sum
@pytest.mark.parametrize("d,f,img,txt,erf,fetching", [(1024, 4096, 6000, 256, False, {"qkv 192x256", "out 128x256", "down 128x256"}),
                                                      (1536, 6144, 1320, 70, False, {"qkv 128x256", "up 192x256", "down 128x256 in 3 parts"}),
                                                      (1536, 6144, 6000, 256, False, {"out 192x256", "down 192x256"}),
                                                      (2048, 10240, 1320, 70, True, {"qkv 192x256", "up 128x256", "down 192x256 in 3 parts"})])
def test_two_streams(d, f, img, txt, erf, fetching):
    """Both streams of a double-stream block in one launch per layer, as the kernel times say, with the weights in one buffer and cut
    between two at several places; right against the oracle, and the same bits wherever they are cut."""
    cfg = wl.BlockConfig("idle_pair", wl.KIND_DOUBLE, n_blocks=2, d=d, n_heads=d // 128, head_dim=128, f=f, n_total=img + txt, n_txt=txt, qk_rmsnorm=True,
                         n_chunks=9, gelu_erf=erf)
    layers = list(paired_layers(cfg))
    assert {f"{n} {t}" + (f" in {p} parts" if p > 1 else "") for n, t, p, on in layers if on} == fetching
    params, inputs = wl.gen_block_params(cfg, 0), wl.gen_block_inputs(cfg, 0)
    run = BlockRunner(cfg)
    want = None
    try:
        for b in range(2):
            run.register_params(b, params)
        t = run.make_io(inputs)
        io = run.io_struct(t)
        for r in (1.0, 0.85, 0.6, 0.3):
            run.ctx.set_resident_fraction(r)
            run.begin(0)
            for i in range(4):                     # each block's weights land before the one ahead of it runs: from the third on one wait
                run.begin((i + 1) % 2)             # for all chunks, and every layer is launched whole, its weights partly in either buffer
                torch.cuda.synchronize()
                if i == 3:
                    run.ctx.cf_kernel_times_reset()
                    run.ctx.cf_set_profiling(True)
                run.fwd(i % 2, io)
                run.ctx.cf_sync()
            times = {k["name"]: k["launches"] for k in run.ctx.cf_kernel_times() if k["launches"]}
            run.ctx.cf_set_profiling(False)
            for name, tile, _, _ in layers:
                assert times.get(f"gemm_{name}/{tile}") == 1 and sum(v for k, v in times.items() if k.startswith(f"gemm_{name}/")) == 1, (r, times)
            got = np.concatenate([t["y_txt"].cpu().numpy(), t["y"].cpu().numpy()])
            want = got if want is None else want
            assert np.array_equal(got.view(np.uint8), want.view(np.uint8)), r
            run.fwd(0, io)                         # the block that was begun
            run.ctx.cf_sync()
    finally:
        run.close()
    rows = np.sort(np.random.default_rng(img).choice(img + txt, 150, replace=False))
    ref = ob.block_forward(cfg, params, inputs, rows=rows)["y_rows"]
    assert rel_l2(want[rows], ref) <= 1e-2
