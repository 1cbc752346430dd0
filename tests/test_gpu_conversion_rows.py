"""Moving fields between the caller's arrays and the workspace: rows of any
length, padded and not, and arrays that start at any element (a snapshot: at
any byte)."""
import numpy as np
import pytest

import oracle
from synth import COURANT, smooth_random

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

H, DT = 10.0, COURANT * 10.0 / 4500.0


def _at(t, offset):
    """A contiguous copy of t whose first element lies `offset` elements past an aligned address."""
    buf = torch.empty(t.numel() + offset, dtype=t.dtype, device=t.device)
    buf[offset:] = t.reshape(-1)
    return buf[offset:].view(t.shape)


@pytest.mark.parametrize("nx", [1, 3, 4, 31, 33, 34, 35, 36, 63, 258])
@pytest.mark.parametrize("storage,bits", [("f32", 32), ("f16", 32), ("bf16", 16)])
@pytest.mark.parametrize("offset", [0, 1])
def test_fields_in_and_out(nx, storage, bits, offset):
    from paper_2404_04441_amd import Solver

    shape = (5, 19, nx)
    print(f"case: nx {nx} {storage} m{bits} offset {offset}", flush=True)
    vel = _at(torch.from_numpy(smooth_random(shape, seed=13)).cuda(), offset)
    s = Solver(vel, H, DT, storage=storage, model_bits=bits, sponge_width=2, sponge_alpha=0.1, tune=False)
    gen = np.random.default_rng(nx)
    second = 1 if storage == "f32" else 2
    # integers below 2^7: exact in every storage
    a, v = (_at(torch.from_numpy(gen.integers(-127, 128, shape).astype(np.float32)).cuda(), offset) for _ in range(2))
    s.write_field(0, a)
    s.write_field(second, v)
    out = _at(torch.full(shape, 7.0, device="cuda"), offset)
    assert torch.equal(s.read_field(0, out), a) and torch.equal(s.read_field(second, out), v)
    if storage != "f32":  # (A - V) / g: the difference is exact; g and the quotient round four times
        want = (a - v).cpu().numpy().astype(np.float64) / oracle.sponge_field(shape, 2, 0.1)
        got = s.read_field(1, out).cpu().numpy()
        assert (np.abs(got - want) <= 5 * 2.0 ** -24 * np.abs(want)).all()
    snap = s.save_state(torch.zeros_like(s.save_state()))  # the gaps between its sections are not written
    s.step(3)
    want = s.read_field(0), s.read_field(second)
    moved = _at(snap, 3 * offset)
    s.load_state(moved)
    assert torch.equal(s.read_field(0), a) and torch.equal(s.read_field(second), v)
    assert torch.equal(s.save_state(torch.zeros_like(moved))[512:], snap[512:])
    s.step(3)
    assert torch.equal(s.read_field(0), want[0]) and torch.equal(s.read_field(second), want[1])
    # the model came in whole: one step from the fields against the oracle's
    if storage == "f32":
        s.load_state(snap)
        s.step(1)
        A, P, V = (t.cpu().numpy().astype(np.float64) for t in (a, v, vel))
        G = oracle.sponge_field(shape, 2, 0.1)
        ref = G * (2 * A - G * P + (V * DT) ** 2 * oracle.laplacian(A, H))
        got = s.read_field(0).cpu().numpy()
        assert np.abs(got - ref).max() <= 1e-6 * np.abs(ref).max()
    s.close()
