"""CPML row and slab kernels: lane widths, ragged bundles and segments, against
the FP64 oracle at the float32 tolerance of the solver (1e-5)."""
import numpy as np
import pytest

import oracle
from oracle.cpml import forward_cpml
from synth import COURANT, ricker, smooth_random

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("shape,W", [
    ((21, 30, 48), 8),     # four-node lanes on rows and slabs; a last bundle of two rows
    ((22, 27, 46), 6),     # two-node lanes; a last bundle of three rows
    ((20, 17, 44), 7),     # four-node rows, one-node slabs (W odd)
    ((19, 25, 45), 9),     # one-node lanes; nz = 2 W + 1: one plane between the z layers
    ((18, 18, 264), 9),    # rows of two segments; no row between the layers
])
def test_layers_match_the_oracle(shape, W):
    from paper_2404_04441_amd import Solver

    nz, ny, nx = shape
    vel = smooth_random(shape, seed=71)
    dt, nt = COURANT * 10.0 / 4500.0, 50
    wav = ricker(nt, dt, 40.0)
    src = (nx // 2, ny // 2, 3)
    rec = np.array([(x, y, 2) for y in range(0, ny, 3) for x in range(0, nx, 4)], dtype=np.int32)
    ref = forward_cpml(vel, 10.0, dt, src, wav, rec, nt, width=W, f0=30.0)
    print(f"case: {shape} W {W}", flush=True)
    s = Solver(torch.from_numpy(vel).cuda(), 10.0, dt, src=src, rec=rec, cpml_width=W, cpml_f0=30.0, tune=False)
    tr = s.run(nt, torch.from_numpy(wav).cuda())
    u = s.read_field(0)
    assert oracle.rel_l2(u.cpu().numpy(), ref["u"]) <= 1e-5
    assert oracle.rel_l2(tr.cpu().numpy(), ref["traces"]) <= 1e-5
    s.close()
