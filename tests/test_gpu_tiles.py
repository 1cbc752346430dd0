"""2.5D tiles of every width and height, on grids that several of them span.

Every tile shape performs the same operations per node, so the results are
compared bit for bit with the 64-wide one-node-per-lane shape's, and that one
with the FP64 oracle.
"""
import numpy as np
import pytest

import oracle
from synth import COURANT, ricker, smooth_random

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _run(vel, dt, wav, src, rec, nt, **kw):
    from paper_2404_04441_amd import Solver

    s = Solver(torch.from_numpy(vel).cuda(), 10.0, dt, src=src, rec=rec, sponge_width=5, sponge_alpha=0.05, **kw)
    tr = s.run(nt, torch.from_numpy(wav).cuda())
    out = s.read_field(0).cpu().numpy(), tr.cpu().numpy()
    s.close()
    return out


@pytest.mark.parametrize("storage,bits", [("f32", 32), ("f16", 32), ("bf16", 16)])
def test_tiles_of_every_width_across_their_edges(storage, bits):
    """nx = 404: two to seven tiles of 64 to 320 nodes with a ragged last one;
    ny = 70 likewise in y; chunks of 1 and 4 planes and one whole chunk (the
    loads past a chunk's end return nothing).  The source sits on a tile
    corner, the receivers are a box across the edges."""
    from paper_2404_04441_amd import variant_count, variant_info

    shape, nt = (11, 70, 404), 24
    vel = smooth_random(shape, seed=11)
    dt = COURANT * 10.0 / 4500.0
    wav = ricker(nt, dt, 60.0)
    src = (320, 32, 5)
    rec = np.array([(x, y, 3) for y in range(0, 70, 3) for x in range(1, 404, 2)], dtype=np.int32)
    base = _run(vel, dt, wav, src, rec, nt, storage=storage, model_bits=bits, variant=7, zchunk=0)
    if storage == "f32":
        ref = oracle.forward(vel, 10.0, dt, src, wav, rec, nt=nt, sponge_width=5, sponge_alpha=0.05)
        assert oracle.rel_l2(base[0], ref["u"]) <= 1e-5 and oracle.rel_l2(base[1], ref["traces"]) <= 1e-5
    assert np.abs(base[0]).max() > 0
    for v in range(1, variant_count()):
        if variant_info(v)["family"] != 0:
            continue
        for zc in (1, 4, 0):
            print(f"case: {storage} m{bits} variant {v} zchunk {zc}", flush=True)
            got = _run(vel, dt, wav, src, rec, nt, storage=storage, model_bits=bits, variant=v, zchunk=zc)
            assert np.array_equal(got[0], base[0]) and np.array_equal(got[1], base[1]), (v, zc)
