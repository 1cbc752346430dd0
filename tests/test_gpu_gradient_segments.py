"""The gradient however its run is cut into segments.

Every second adjoint step updates the image with two terms, the last one with
one, and a term may wait across a segment's start: the sums keep their order,
so every checkpoint interval gives the same bits."""
import numpy as np
import pytest

import oracle
from oracle import adjoint as oadj
from synth import COURANT, ricker, smooth_random

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("nt", [1, 2, 3, 8, 13])
@pytest.mark.parametrize("nx,rec_kind", [(40, "box"), (37, "list")])
def test_every_interval_gives_the_same_gradient(nt, nx, rec_kind):
    from paper_2404_04441_amd import Solver

    shape = (14, 18, nx)
    vel = smooth_random(shape, seed=23)
    dt = COURANT * 10.0 / 4500.0
    wav = ricker(nt, dt, 100.0, t0=3 * dt)
    src = (nx // 2, 9, 6)
    gen = np.random.default_rng(nt)
    if rec_kind == "box":  # the source's node among them: nt = 2 has a gradient already
        rec = np.array([(x, y, 6) for y in range(5, 14) for x in range(10, 30)], dtype=np.int32)
    else:
        rec = np.stack([gen.integers(nx // 2 - 6, nx // 2 + 6, 60), gen.integers(3, 15, 60), gen.integers(2, 12, 60)], 1).astype(np.int32)
    resid = gen.standard_normal((nt, len(rec))).astype(np.float32)
    ref, _, _ = oadj.gradient(vel, 10.0, dt, src, wav, rec, nt, resid=resid.astype(np.float64), sponge_width=3,
                              sponge_alpha=0.05)
    grads = []
    for K in sorted({1, 2, 3, 5, nt, 0}):
        print(f"case: nt {nt} nx {nx} {rec_kind} interval {K}", flush=True)
        s = Solver(torch.from_numpy(vel).cuda(), 10.0, dt, src=src, rec=rec, sponge_width=3, sponge_alpha=0.05,
                   adjoint=True, nt_max=nt, ckpt_interval=min(K, nt), tune=False)
        for _ in range(2):  # a second call starts from the first one's leftovers
            grads.append(s.adjoint(nt, torch.from_numpy(wav).cuda(), torch.from_numpy(resid).cuda()).cpu().numpy())
        s.close()
    for g in grads[1:]:
        assert np.array_equal(g, grads[0])
    if nt > 1:
        assert np.abs(ref).max() > 0 and oracle.rel_l2(grads[0], ref) <= 1e-4
    else:
        assert not grads[0].any()
