"""The forms in which a block launches attention, each asked for by name (cf_op_attention_form): keys in parts that a second
kernel merges, sweeps dealt out by the kernel in even shares or drawn from a counter."""
import numpy as np
import pytest
import torch

from paper_2605_11335_amd import binding as B
from tests.util import bf16_round, bits_to_f64, dev_bits, host_bits, max_abs, rel_l2

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
FLAG_BYTES = 4096


def operands(q, k, v):
    """bf16 operands on the device as the kernel takes them, and the rounded values."""
    H, nk, hd = k.shape
    pad = (nk + 63) // 64 * 64
    (qf, qb), (kf, kb), (vf, vb) = bf16_round(q), bf16_round(k), bf16_round(v)
    vt = np.zeros((H, hd, pad), np.uint16)
    vt[:, :, :nk] = vb.transpose(0, 2, 1)
    return (dev_bits(qb), dev_bits(kb), dev_bits(vt), H, q.shape[1], nk, pad, hd), (qf, kf, vf)


def form(ops, parts=1, all_parts=False, deal=0, no_wait=False):
    q, k, vt, H, nq, nk, pad, hd = ops
    floats = parts * H * ((nq + 31) // 32) * 32 * (hd + 2) if parts > 1 else 24 * 32 * 512 * 66
    scratch = torch.full((FLAG_BYTES // 4 + floats,), float("nan"), device=DEV)
    scratch[:FLAG_BYTES // 4] = 0.0
    o = torch.zeros((H, nq, hd), dtype=torch.int16, device=DEV)
    B.cf_op_attention_form(q, k, vt, o, H, nq, nk, pad, hd, None if all_parts else scratch, parts, all_parts, deal, no_wait)
    torch.cuda.synchronize()
    return host_bits(o)


def whole(ops):
    """Sweeps over all keys by the grid's workgroups, which cf_op_attention need not take (few queries)."""
    return form(ops)


def reference(values):
    q, k, v = (a.astype(np.float64) for a in values)
    out = np.empty_like(q)
    for h in range(q.shape[0]):
        s = q[h] @ k[h].T / np.sqrt(q.shape[2])
        p = np.exp(s - s.max(1, keepdims=True))
        out[h] = (p / p.sum(1, keepdims=True)) @ v[h]
    return out


# parts that end inside, at and one key past a tile; a last part of one ragged tile; workgroups of 4, 7 and 8 waves
@pytest.mark.parametrize("H,nq,nk,hd,parts", [(1, 1888, 1888, 64, 5), (2, 77, 2265, 64, 6), (3, 300, 513, 64, 3), (1, 33, 449, 128, 4),
                                              (3, 1000, 1153, 128, 4), (2, 4500, 640, 128, 2), (8, 3500, 9000, 64, 2),
                                              (1, 27000, 17000, 128, 2), (1, 27000, 34000, 128, 2), (1, 27000, 34000, 64, 2)])
@pytest.mark.parametrize("sharp", [1.0, 24.0])
def test_keys_in_parts(H, nq, nk, hd, parts, sharp):
    rng = np.random.default_rng(nq + nk + hd + parts)
    q, k, v = (rng.normal(size=(H, n, hd)) for n in (nq, nk, nk))
    ops, values = operands(q * np.sqrt(sharp), k * np.sqrt(sharp), v)
    got = bits_to_f64(form(ops, parts=parts))
    # also where the two forms differ in the height of a workgroup, and with it in the sweeps that are repeated for scores out of range
    assert np.array_equal(form(ops, parts=parts, all_parts=True), form(ops, parts=parts))
    rows = np.sort(rng.choice(nq, min(nq, 600), replace=False))
    ref = reference((values[0][:, rows], values[1], values[2]))
    print(f"rel_l2={rel_l2(got[:, rows], ref):.3e} max_abs={max_abs(got[:, rows], ref):.3e}", flush=True)
    assert rel_l2(got[:, rows], ref) < 6e-3 and max_abs(got[:, rows], ref) < 2e-2 * max(1.0, np.abs(ref).max())


# groups of 32 query tiles: 8 and a quarter, 9 exactly, 9 and a quarter; key counts of 75, 43, 5 and 4 tiles, ragged
@pytest.mark.parametrize("H,nq,nk", [(12, 4800, 4800), (24, 2850, 2750), (11, 6800, 300), (12, 4800, 200)])
@pytest.mark.parametrize("deal", [1, 2])
def test_dealt_out_sweeps_have_the_bits_of_whole_ones(H, nq, nk, deal):
    """Also where no workgroup ever finds the state that another left, and starts its sweep over."""
    rng = np.random.default_rng(nq + nk)
    ops, _ = operands(*(rng.normal(size=(H, n, 128)) for n in (nq, nk, nk)))
    want = whole(ops)
    for no_wait in (False, True):
        assert np.array_equal(form(ops, deal=deal, no_wait=no_wait), want), no_wait


# the scores of half of the heads leave the range of a sweep without a running maximum at one tile: in the first piece of a cut
# sweep, in any later one, at the very end
@pytest.mark.parametrize("H,nq,nk", [(12, 8400, 2030), (12, 4700, 2030), (12, 4800, 4800)])      # 13 groups, eighths cut inside; 8, in pieces if drawn
@pytest.mark.parametrize("at", [0.02, 0.2, 0.4, 0.6, 0.8, 0.99])
@pytest.mark.parametrize("deal", [1, 2])
def test_dealt_out_sweeps_that_have_to_be_repeated(H, nq, nk, at, deal):
    """A cut sweep is then repeated from its first tile, as a whole one is, whichever of its pieces found out."""
    assert B.cf_plan_attention(H, nq, nk, 128) == 8            # the height of the dealt out sweeps
    rng = np.random.default_rng(nk)
    q, k, v = (rng.normal(size=(H, n, 128)) for n in (nq, nk, nk))
    u = rng.normal(size=128)
    u /= np.linalg.norm(u)
    q += 4.0 * u
    jump = int(at * nk) // 64 * 64
    k[::2, jump:jump + 64] += 600.0 * u                        # 4 * 600 / sqrt(128) = 212 nats
    ops, values = operands(q, k, v)
    want = whole(ops)
    rows = np.sort(rng.choice(nq, 100, replace=False))
    got, ref = bits_to_f64(want)[:, rows], reference((values[0][:, rows], values[1], values[2]))
    assert rel_l2(got, ref) < 6e-3
    for no_wait in (False, True):
        out = form(ops, deal=deal, no_wait=no_wait)
        assert np.array_equal(out, want), (no_wait, int((out != want).sum()))


@pytest.mark.parametrize("hd,parts,all_parts", [(64, 1, 0), (64, 3, 0), (64, 3, 1), (64, 3, 2), (128, 1, 0), (128, 3, 0), (128, 3, 1), (128, 3, 2)])
def test_a_sample_has_the_same_bits_alone_and_in_a_batch(hd, parts, all_parts):
    """Scores with a standard deviation of 24 leave the fast softmax's range for some waves of 32 queries and not for others.  A
    workgroup repeats its sweep if one of its waves has to, and there are more waves in it where a batch fills the chip: those
    in range keep their bits."""
    H, nq, nk, batch = 2, 2300, 2000, 14
    assert B.cf_plan_attention(H, nq, nk, hd) == 4 and B.cf_plan_attention(batch * H, nq, nk, hd) > 4
    rng = np.random.default_rng(hd)
    q, k, v = (rng.normal(size=(H, n, hd)) * s for n, s in ((nq, 24.0 ** 0.5), (nk, 24.0 ** 0.5), (nk, 1.0)))
    ops, _ = operands(q, k, v)
    many = tuple(t.repeat((batch,) + (1,) * (t.dim() - 1)) for t in ops[:3]) + (batch * H,) + ops[4:]
    alone = form(ops, parts=parts, all_parts=all_parts)
    for got in form(many, parts=parts, all_parts=all_parts).reshape(batch, H, nq, hd):
        assert np.array_equal(got, alone), int((got != alone).sum())
    # of a sample's parts it does not matter who sweeps them
    if parts > 1:
        assert np.array_equal(form(ops, parts=parts), alone)
