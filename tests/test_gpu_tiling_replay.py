"""A choice made on padded rows is reported as a variant that asks for padded
rows: passed back, it gives the same layout, not only the same tiles."""
import numpy as np
import pytest

from synth import COURANT, ricker, smooth_random

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("storage", ["f32", "f16"])
def test_padded_layout_survives_the_round_trip(storage):
    """nx = 70: every padded form, of one, two and four nodes per lane, and the
    library's own choices."""
    from paper_2404_04441_amd import Solver, variant_count, variant_info

    shape, nt = (13, 17, 70), 20
    vel = torch.from_numpy(smooth_random(shape, seed=31)).cuda()
    dt = COURANT * 10.0 / 4500.0
    wav = torch.from_numpy(ricker(nt, dt, 50.0)).cuda()
    rec = np.array([(x, 8, 4) for x in range(70)], dtype=np.int32)

    def solver(**kw):
        return Solver(vel, 10.0, dt, src=(67, 8, 6), rec=rec, sponge_width=4, sponge_alpha=0.05, storage=storage, **kw)

    plain = solver(variant=7)
    want = plain.run(nt, wav), plain.read_field(0)
    choices = [dict(tune=False), dict(tune=True)]
    families = set()
    for v in range(29, variant_count()):  # the padded forms
        if storage == "f32" or variant_info(v)["family"] == 0:
            choices.append(dict(variant=v))
            families.add(variant_info(v)["family"])
    assert families == ({0, 1, 2} if storage == "f32" else {0})
    for kw in choices:
        print(f"case: {storage} {kw}", flush=True)
        a = solver(**kw)
        assert a.workspace_bytes > plain.workspace_bytes
        if "variant" in kw:
            assert a.tiling()["variant"] == kw["variant"]
        b = solver(tune=False, **a.tiling())
        assert b.tiling() == a.tiling() and b.workspace_bytes == a.workspace_bytes
        for s in (a, b):
            assert torch.equal(s.run(nt, wav), want[0]) and torch.equal(s.read_field(0), want[1])
            s.close()
    plain.close()
