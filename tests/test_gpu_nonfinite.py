"""Infinities, NaN and values at the ends of the fp32 range: what comes out of a kernel where they go in."""
import numpy as np
import pytest
import torch

import workload as wl
from paper_2605_11335_amd import binding as B
from tests.test_gpu_attention_forms import form, operands, reference, whole
from tests.util import bits_to_f64, host_bits, max_abs, rel_l2

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("erf", [False, True])
def test_activation_at_the_ends_of_the_range(erf):
    """Pre-activations handed in as the bias of a layer over zeros.  GELU tends to the identity on the right and to zero on the
    left, so +inf and every value past 20 come through and what lies below -20 is zero; NaN stays NaN."""
    vals = np.array([np.inf, 3.0e38, 1.0e30, 4.0e19, 1000.0, 20.5, 20.0, 19.5, 13.0, 0.0, -20.5, -1000.0, -4.0e19, -3.0e38, np.nan, 1.0],
                    np.float32)
    bits = wl.f32_to_bf16_bits(vals)
    z = bits_to_f64(bits)
    M, N, K = 70, len(vals), 64
    buf = np.zeros(2 * N * K + 2 * N, np.uint8)
    buf[2 * N * K:] = bits.view(np.uint8)
    blob = torch.from_numpy(buf).to(DEV)
    out = torch.zeros((M, N), dtype=torch.int16, device=DEV)
    B.cf_op_linear(torch.zeros((M, K), dtype=torch.int16, device=DEV), blob, 0, 2 * N * K, M, N, K, None, out, n_split=0, gelu_erf=erf)
    torch.cuda.synchronize()
    got = bits_to_f64(host_bits(out))
    assert np.array_equal(got, np.broadcast_to(got[0], got.shape), equal_nan=True)
    for v, g in zip(z, got[-1]):
        if np.isnan(v):
            assert np.isnan(g)
        elif v >= 13.0:
            assert g == v, (v, g)
        elif v <= -20.0 or v == 0.0:
            assert g == 0.0, (v, g)
    assert abs(got[-1][-1] - 0.8413447) < 2.0 ** -8


# the first tile of the sequence, of each part in turn, of a part that holds no other key, the last (ragged) tile, and all but one
@pytest.mark.parametrize("hd", [64, 128])
@pytest.mark.parametrize("parts", [1, 2, 3, 5])
@pytest.mark.parametrize("lo,hi", [(0, 64), (0, 192), (192, 256), (256, 384), (320, 384), (384, 448), (512, 577), (64, 577)])
def test_tiles_of_scores_of_minus_infinity(hd, parts, lo, hi):
    """Keys whose scores are all -inf have a weight of zero, wherever they lie."""
    H, nq, nk = 2, 300, 577
    rng = np.random.default_rng(hd + parts + lo)
    q, k, v = (rng.normal(size=(H, n, hd)) for n in (nq, nk, nk))
    q[:, :, 0] = np.abs(q[:, :, 0]) + 0.5
    ops, values = operands(q, k, v)
    ops[1][:, lo:hi, 0] = -128                     # the bits of -inf in bf16: 0xff80
    got = bits_to_f64(whole(ops) if parts == 1 else form(ops, parts=parts))
    values[1][:, lo:hi, 0] = -np.inf
    ref = reference(values)
    assert np.isfinite(ref).all() and np.isfinite(got).all()
    if parts > 1:
        for all_parts in (1, 2) if parts <= (8 if hd == 64 else 4) else (1,):      # one after the other, a wave to each
            assert np.array_equal(form(ops, parts=parts, all_parts=all_parts), form(ops, parts=parts)), all_parts
    print(f"rel_l2={rel_l2(got, ref):.3e}", flush=True)
    assert rel_l2(got, ref) < 6e-3 and max_abs(got, ref) < 2e-2 * max(1.0, np.abs(ref).max())
