"""A run that diverged is recovered by restoring a snapshot or by setting both
stored levels anew, as well as by a reset: nothing of the non-finite field
stays in the workspace, in the columns that pad its rows either."""
import numpy as np
import pytest

from synth import COURANT, smooth_random

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("nx", [68, 70, 71])  # rows padded by no column, two and one
@pytest.mark.parametrize("storage", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("how", ["load_state", "write_field"])
def test_recovery_from_a_nonfinite_field(nx, storage, how):
    from paper_2404_04441_amd import Solver

    shape = (13, 17, nx)
    vel = torch.from_numpy(smooth_random(shape, seed=83)).cuda()
    rec = np.array([(x, y, 4) for y in range(17) for x in range(nx)], dtype=np.int32)
    print(f"case: nx {nx} {storage} {how}", flush=True)
    s = Solver(vel, 10.0, COURANT * 10.0 / 4500.0, rec=rec, sponge_width=4, sponge_alpha=0.05, storage=storage, tune=False)
    second = 1 if storage == "f32" else 2
    gen = np.random.default_rng(5)
    fields = [torch.from_numpy((k * gen.standard_normal(shape)).astype(np.float32)).cuda() for k in (1.0, 0.05)]

    def set_fields():
        s.write_field(0, fields[0])
        s.write_field(second, fields[1])

    set_fields()
    snap = s.save_state()
    want = s.step(8)[:8].clone(), s.read_field(0), s.read_field(1)
    for value in (float("nan"), float("inf")):
        s.write_field(0, torch.full(shape, value, device="cuda"))
        s.step(3)
        assert not torch.isfinite(s.read_field(0)).any()
        if how == "load_state":
            s.load_state(snap)
        else:
            set_fields()
        n = s.time_index()
        got = s.step(8)[n:n + 8], s.read_field(0), s.read_field(1)
        assert s.sync_status() == 0
        for a, b in zip(got, want):
            assert torch.equal(a, b)
    s.close()
