"""16-bit storage: the scale bookkeeping of the step.

The step works in the stored units, with the scales folded into its factors;
fields whose exponents lie far apart go through a path of their own.  The
maxima that fix the next exponents come from per-level slots that every
workgroup raises.
"""
import numpy as np
import pytest

import oracle
from oracle.storage import growth_bound_gamma, quantize, scale_exponent
from synth import COURANT, ricker, smooth_random

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

SHAPE, H = (19, 23, 72), 10.0
ULP = {"f16": 2.0 ** -10, "bf16": 2.0 ** -7}
TINY = {"f16": 2.0 ** -24, "bf16": 2.0 ** -133}


def _solver(fmt, nt=8, **kw):
    from paper_2404_04441_amd import Solver

    vel = smooth_random(SHAPE, seed=61)
    dt = COURANT * H / 4500.0
    wav = ricker(nt, dt, 60.0)
    rec = np.array([(x, 11, 7) for x in range(0, 72, 5)], dtype=np.int32)
    s = Solver(torch.from_numpy(vel).cuda(), H, dt, src=(33, 12, 9), rec=rec, sponge_width=4, sponge_alpha=0.05,
               storage=fmt, **kw)
    return s, vel, dt, wav, rec


def _terms(u):
    c = oracle.second_derivative_weights(4)
    P = np.pad(u, 4)
    out = np.zeros_like(u)
    for axis in range(3):
        for m in range(1, 5):
            for k in (m, -m):
                sl = [slice(4, -4)] * 3
                sl[axis] = slice(4 + k, P.shape[axis] - 4 + k)
                out += abs(c[m]) / H ** 2 * (np.abs(P[tuple(sl)]) + np.abs(u))
    return out


@pytest.mark.parametrize("fmt,a_size,v_size", [("f16", 1e9, 1e-7), ("bf16", 1e-9, 1e8), ("f16", 3.0, 0.1),
                                               ("bf16", 0.0, 1e-12), ("f16", 1e25, 1e-25)])
def test_one_step_at_any_pair_of_scales(fmt, a_size, v_size):
    """One step from a random state whose fields differ in size by up to 50
    decades, against the oracle's float64 step rounded at the rule's
    exponents: each stored value within one unit of the format's last place
    plus 16 float32 roundings of the size of its terms (the evaluation bound)."""
    s, vel, dt, wav, rec = _solver(fmt, tune=False)
    gen = np.random.default_rng(5)
    print(f"case: {fmt} A {a_size} V {v_size}", flush=True)
    s.reset()
    s.write_field(0, torch.from_numpy((a_size * gen.standard_normal(SHAPE)).astype(np.float32)).cuda())
    s.write_field(2, torch.from_numpy((v_size * gen.standard_normal(SHAPE)).astype(np.float32)).cuda())
    A, V = (s.read_field(k).cpu().numpy().astype(np.float64) for k in (0, 2))
    tr = s.step(1, torch.from_numpy(wav).cuda())
    got = {0: s.read_field(0).cpu().numpy().astype(np.float64), 2: s.read_field(2).cpu().numpy().astype(np.float64)}
    s.close()
    G = oracle.sponge_field(SHAPE, 4, 0.05)
    M = (dt * vel.astype(np.float64)) ** 2
    q = np.zeros(SHAPE)
    q[9, 12, 33] = dt * dt * float(wav[0]) / H ** 3
    vn = G * (V + M * oracle.laplacian(A, H) + q)
    an = G * A + vn
    tv = G * (np.abs(V) + M * _terms(A) + np.abs(q))
    bv = np.abs(V).max() + growth_bound_gamma(float(vel.max()), H, dt) * np.abs(A).max() + np.abs(q).max()
    for which, want, terms, e in ((0, an, G * np.abs(A) + tv, scale_exponent(np.abs(A).max() + bv)),
                                  (2, vn, tv, scale_exponent(bv))):
        stored = got[which] * 2.0 ** e
        assert np.isfinite(stored).all() and np.array_equal(quantize(stored, fmt), stored)
        emu = quantize(want * 2.0 ** e, fmt)
        step = np.maximum(ULP[fmt] * np.abs(emu), TINY[fmt])
        # float32 results below its normal range may flush
        bound = step + 16 * 2.0 ** -24 * terms * 2.0 ** e + 2.0 ** -100 * 2.0 ** e
        assert (np.abs(stored - emu) / bound).max() <= 1.0, which
    assert np.array_equal(tr.cpu().numpy()[0], got[0][rec[:, 2], rec[:, 1], rec[:, 0]].astype(np.float32))


@pytest.mark.parametrize("fmt", ["f16", "bf16"])
def test_maxima_of_an_earlier_field_do_not_linger(fmt):
    """Setting fields of another size in the middle of a run gives the bits of
    a context that starts with them at the same step: no slot keeps a maximum of
    the field that was replaced.  Replays from graphs keep the records too."""
    gen = np.random.default_rng(7)
    big, small = (torch.from_numpy((k * gen.standard_normal(SHAPE)).astype(np.float32)).cuda() for k in (1e4, 1e-3))
    outs = []
    for first, kw in ((True, {}), (False, {}), (True, {"graph_steps": 2})):
        s, _, _, wav, _ = _solver(fmt, nt=12, **kw)
        wav = torch.from_numpy(wav).cuda()
        s.reset()
        if first:
            s.write_field(0, big)
            s.write_field(2, big)
            s.step(4, wav)
        else:
            s.step(4, wav)
        s.write_field(0, small)
        s.write_field(2, small)
        s.step(6, wav)
        outs.append([s.read_field(k).cpu().numpy() for k in (0, 2)])
        s.close()
    for o in outs[1:]:
        assert np.array_equal(o[0], outs[0][0]) and np.array_equal(o[1], outs[0][1])
