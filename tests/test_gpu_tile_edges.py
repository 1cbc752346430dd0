"""Full-size grids across the edges of the tiles that run on them, whatever
their width: sampled there against the oracle, and whole fields bit for bit
against a one-node-per-lane shape of another tile."""
import numpy as np
import pytest

import oracle
from synth import COURANT

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

H, DT = 10.0, COURANT * 10.0 / 4500.0


def _state(shape, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    vel = 1500.0 + 3000.0 * torch.rand(shape, generator=gen, device="cuda")
    return vel, torch.randn(shape, generator=gen, device="cuda"), 0.05 * torch.randn(shape, generator=gen, device="cuda")


def _step(vel, a, b, storage, **kw):
    from paper_2404_04441_amd import Solver

    s = Solver(vel, H, DT, src=(5, 6, 7), sponge_width=20, storage=storage, **kw)
    s.write_field(0, a)
    s.write_field(1 if storage == "f32" else 2, b)
    s.step(1, torch.full((1,), 1e8, device="cuda"))
    out = s.read_field(0), s.read_field(1 if storage == "f32" else 2)
    tiling = s.tiling()
    s.close()
    return out, tiling


class _Nodes:
    """The values of a field at the nodes asked for, as field[z, y, x]."""

    def __init__(self, field, nodes):
        k = torch.tensor(sorted(nodes), device="cuda")
        self.shape = tuple(field.shape)
        self.at = dict(zip(map(tuple, k.tolist()), field[k[:, 0], k[:, 1], k[:, 2]].double().tolist()))

    def __getitem__(self, zyx):
        return self.at[zyx]


@pytest.mark.parametrize("shape,kw", [
    ((96, 384, 384), dict(tune=True)), ((60, 300, 404), dict(tune=True)),
    *[((40, 128, 960), dict(variant=v)) for v in (20, 22, 24, 26, 27, 28)]])
def test_both_sides_of_every_tile_edge(shape, kw):
    from paper_2404_04441_amd import variant_tile

    vel, a, b = _state(shape, 5)
    (new, _), tiling = _step(vel, a, b, "f32", **kw)
    tx, ty = variant_tile(tiling["variant"])
    print(f"case: {shape} {tiling} tile {tx} x {ty}", flush=True)
    nz, ny, nx = shape

    def around(step, n):
        k = np.arange(step, n, step)
        return np.concatenate([k - 1, k, k - 4, np.minimum(k + 3, n - 1), [0, 1, 3, 4, 19, 20, n - 1, n - 4, n - 5]])

    rng = np.random.default_rng(6)
    pts = np.stack([rng.choice(around(tx, nx), 2000), rng.choice(around(ty, ny), 2000),
                    rng.choice(around(tiling["zchunk"], nz), 2000)], 1)
    need = {(z + c * (k == 2), y + c * (k == 1), x + c * (k == 0)) for x, y, z in pts.tolist() for k in range(3)
            for c in range(-4, 5)}
    need = {n for n in need if all(0 <= i < m for i, m in zip(n, shape))}
    ref = oracle.step_at(pts, _Nodes(a, need), _Nodes(b, need), _Nodes(vel, need), H, DT, src=(5, 6, 7), s_n=1e8,
                         sponge_width=20, sponge_alpha=0.015)
    p = torch.from_numpy(pts).cuda()
    got = new[p[:, 2], p[:, 1], p[:, 0]].double().cpu().numpy()
    assert np.abs(got - ref).max() <= 1e-6 * float(new.abs().max())


@pytest.mark.parametrize("n,storage,bits", [(512, "f32", 32), (768, "f32", 32), (512, "f16", 32), (512, "f16", 16),
                                            (512, "bf16", 32), (1024, "bf16", 16), (1024, "f16", 16)])
def test_the_tuned_choice_gives_the_bits_of_another_tile(n, storage, bits):
    vel, a, b = _state((n, n, n), n)
    got, tiling = _step(vel, a, b, storage, model_bits=bits, tune=True)
    print(f"case: {n} {storage} m{bits} {tiling}", flush=True)
    want, _ = _step(vel, a, b, storage, model_bits=bits, variant=7)
    assert torch.isfinite(want[0]).all() and float(want[0].abs().max()) > 0
    assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
