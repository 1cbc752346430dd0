"""Half storage with m in 16-bit codes, the form with a Laplacian of its own
(summed from the centre weight): over every tile shape, on padded rows, and with
exponents far apart, where a path of its own has to give the same sums."""
import numpy as np
import pytest

import oracle
import test_gpu_padded_rows as padded
import test_gpu_storage_scales as scales
import test_gpu_tiles as tiles
from oracle.storage import growth_bound_gamma, quantize, scale_exponent

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def test_every_tile():
    tiles.test_tiles_of_every_width_across_their_edges("f16", 16)


@pytest.mark.parametrize("nx", [33, 34, 71, 301])
@pytest.mark.parametrize("rec_kind", ["box", "list"])
def test_padded_rows(nx, rec_kind):
    padded.test_padded_rows_are_bitwise_the_unpadded_ones(nx, rec_kind, "f16", 16)


@pytest.mark.parametrize("a_size,v_size", [(3.0, 0.1), (1e9, 1e-7), (1e-9, 1e8), (1e25, 1e-25)])
def test_one_step_at_any_pair_of_scales(a_size, v_size):
    """Against the oracle's float64 step on the model the codes represent,
    rounded at the rule's exponents: within one unit of the format's last place
    plus 16 float32 roundings of the size of its terms; and bit for bit between
    two tiles."""
    print(f"case: A {a_size} V {v_size}", flush=True)
    gen = np.random.default_rng(15)
    fields = [torch.from_numpy((k * gen.standard_normal(scales.SHAPE)).astype(np.float32)).cuda() for k in (a_size, v_size)]
    outs = []
    for variant in (0, 7):
        s, vel, dt, wav, _ = scales._solver("f16", model_bits=16, tune=False, variant=variant)
        s.reset()
        s.write_field(0, fields[0])
        s.write_field(2, fields[1])
        A, V = (s.read_field(k).cpu().numpy().astype(np.float64) for k in (0, 2))
        s.step(1, torch.from_numpy(wav).cuda())
        outs.append([s.read_field(k).cpu().numpy() for k in (0, 2)])
        s.close()
    assert all(np.array_equal(a, b) for a, b in zip(*outs))
    # the codes as the library forms them: t = v dt, t t - lo in one rounding
    # (an fma) and the quotient in float32, lo and the step from float32 squares
    f = np.float32
    t = vel.astype(f) * f(dt)
    lo, step = t.min() ** 2, (t.max() ** 2 - t.min() ** 2) / f(65535)
    u = np.rint((t.astype(np.float64) ** 2 - float(lo)).astype(f) / step)
    M = np.clip(u, 0, 65535).astype(np.float64) * float(step) + float(lo)
    G = oracle.sponge_field(scales.SHAPE, 4, 0.05)
    q = np.zeros(scales.SHAPE)
    q[9, 12, 33] = dt * dt * float(wav[0]) / scales.H ** 3
    vn = G * (V + M * oracle.laplacian(A, scales.H) + q)
    an = G * A + vn
    tv = G * (np.abs(V) + M * scales._terms(A) + np.abs(q))
    bv = np.abs(V).max() + growth_bound_gamma(float(vel.max()), scales.H, dt) * np.abs(A).max() + np.abs(q).max()
    for got, want, terms, e in ((outs[0][0], an, G * np.abs(A) + tv, scale_exponent(np.abs(A).max() + bv)),
                                (outs[0][1], vn, tv, scale_exponent(bv))):
        stored = got.astype(np.float64) * 2.0 ** e
        assert np.isfinite(stored).all() and np.array_equal(quantize(stored, "f16"), stored)
        emu = quantize(want * 2.0 ** e, "f16")
        ulp = np.maximum(scales.ULP["f16"] * np.abs(emu), scales.TINY["f16"])
        bound = ulp + 16 * 2.0 ** -24 * terms * 2.0 ** e + 2.0 ** -100 * 2.0 ** e
        assert (np.abs(stored - emu) / bound).max() <= 1.0
