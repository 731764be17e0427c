"""Keys in parts with a wave of one workgroup to each (few queries): the bits of the parts that a kernel merges, and right against
a float64 reference; also where scores leave the range of a sweep without a running maximum, or are -inf."""
import numpy as np
import pytest

from tests.test_gpu_attention_forms import form, operands, reference
from tests.util import bits_to_f64, max_abs, rel_l2

pytestmark = pytest.mark.gpu


# one query and a ragged wave of 32; parts of two tiles and more, a last part of one ragged tile, two to eight parts
@pytest.mark.parametrize("H,nq,nk,hd,parts", [(1, 1, 130, 64, 2), (8, 512, 512, 64, 4), (3, 77, 963, 64, 8), (2, 33, 449, 128, 4), (3, 300, 1025, 128, 3),
                                              (1, 2000, 3000, 128, 4), (5, 100, 1900, 64, 5)])
@pytest.mark.parametrize("sharp", [1.0, 24.0])
def test_a_wave_to_each_part(H, nq, nk, hd, parts, sharp):
    rng = np.random.default_rng(nq + nk + hd + parts)
    q, k, v = (rng.normal(size=(H, n, hd)) for n in (nq, nk, nk))
    ops, values = operands(q * np.sqrt(sharp), k * np.sqrt(sharp), v)
    got = form(ops, parts=parts, all_parts=2)
    assert np.array_equal(got, form(ops, parts=parts))         # also where a sweep is repeated for scores out of range
    ref, got = reference(values), bits_to_f64(got)
    assert rel_l2(got, ref) < 6e-3 and max_abs(got, ref) < 2e-2 * max(1.0, np.abs(ref).max())


@pytest.mark.parametrize("hd", [64, 128])
def test_scores_out_of_range(hd):
    rng = np.random.default_rng(5)
    q, k, v = (rng.normal(size=(2, n, hd)) for n in (70, 1000, 1000))
    u = np.ones(hd) / np.sqrt(hd)
    q += 4.0 * u
    k[0, 640:704] += 600.0 * u                                 # 300 or 212 nats above the tiles before it, inside a part
    k[1, :256] = np.where(np.arange(hd) == 0, -np.inf, 0.0)    # a whole part of -inf (or +inf: q < 0) scores
    q[1, :, 0] = np.abs(q[1, :, 0]) + 0.1
    ops, values = operands(q, k, v)
    got = bits_to_f64(form(ops, parts=4, all_parts=2))
    ref = reference((values[0][:1], values[1][:1], values[2][:1]))
    assert rel_l2(got[:1], ref) < 6e-3
    ref = reference((values[0][1:], values[1][1:, 256:], values[2][1:, 256:]))
    assert rel_l2(got[1:], ref) < 6e-3
