"""Receiver lists sampled by the step after: the same traces however a run is cut."""
import numpy as np
import pytest

from synth import COURANT, ricker, smooth_random

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("count", [1, 300, 2000])
@pytest.mark.parametrize("kw", [dict(), dict(storage="f16"), dict(storage="bf16", model_bits=16),
                                dict(cpml_width=6, sponge_width=0)])
def test_lists_are_sampled_alike_however_the_run_is_cut(count, kw):
    """One receiver, more than a workgroup's worth, and more than the grid's
    tiles have threads; whole run, single steps, graph replays with the
    program's own work between them."""
    from paper_2404_04441_amd import Solver

    shape, nt = (17, 21, 53), 23
    vel = torch.from_numpy(smooth_random(shape, seed=91)).cuda()
    dt = COURANT * 10.0 / 4500.0
    wav = torch.from_numpy(ricker(nt, dt, 60.0)).cuda()
    gen = np.random.default_rng(count)
    rec = np.stack([gen.integers(0, n, count) for n in (53, 21, 17)], 1).astype(np.int32)
    opts = dict(src=(26, 10, 8), rec=rec, sponge_width=4, sponge_alpha=0.05)
    opts.update(kw)
    print(f"case: {count} receivers {kw}", flush=True)
    s = Solver(vel, 10.0, dt, tune=False, **opts)
    whole = s.run(nt, wav).clone()
    assert float(whole.abs().max()) > 0
    # each row is the field after its step
    s.reset()
    tr = torch.full((nt, count), float("nan"), device="cuda")
    for n in range(nt):
        s.step(1, wav, tr)
        u = s.read_field(0)
        at = torch.from_numpy(rec.astype(np.int64)).cuda()
        assert torch.equal(tr[n], u[at[:, 2], at[:, 1], at[:, 0]])
    assert torch.equal(tr, whole)
    s.close()
    g = Solver(vel, 10.0, dt, tune=False, graph_steps=4, **opts)
    tr = torch.full((nt, count), float("nan"), device="cuda")
    for _ in range(3):
        g.run(nt, wav, tr)
        torch.cuda.synchronize()
        assert torch.equal(tr, whole)
        tr.fill_(float("nan"))
        torch.cuda.synchronize()
    g.close()
