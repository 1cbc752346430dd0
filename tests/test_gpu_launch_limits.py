"""Grids whose row kernels need more wavefronts than one launch holds (fewer
than 2^32 threads): tens of millions of rows of a node or two."""
import numpy as np
import pytest

from synth import COURANT, ricker

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

H, DT = 10.0, COURANT * 10.0 / 4500.0


def test_previous_level_of_67_million_rows():
    """A^{n-1} = (A^n - V^n) / g of 16-bit storage, row by row: 2^26 rows of one
    node.  Without a sponge g is 1 and the values chosen are exact in f16."""
    from paper_2404_04441_amd import Solver

    shape = (8192, 8192, 1)
    s = Solver(torch.full(shape, 3000.0, device="cuda"), H, DT, storage="f16", tune=False)
    a = torch.randint(-512, 512, shape, device="cuda").float()
    v = torch.randint(-512, 512, shape, device="cuda").float()
    print("case: 1 x 8192 x 8192", flush=True)
    s.write_field(0, a)
    s.write_field(2, v)
    assert torch.equal(s.read_field(1), a - v)
    s.close()


def test_cpml_of_134_million_layer_rows():
    """2 x 2 x 2^26 nodes with layers of one node: every row lies in a y layer.
    The planes around the source, next to the first z layer, are those of a
    grid of 64 planes as long as nothing reaches its end (9 planes a step)."""
    from paper_2404_04441_amd import Solver

    nt = 5
    wav = torch.from_numpy(ricker(nt, DT, 60.0, t0=2 * DT)).cuda()
    out = []
    for nz in (64, 1 << 26):
        print(f"case: 2 x 2 x {nz}", flush=True)
        s = Solver(torch.full((nz, 2, 2), 3000.0, device="cuda"), H, DT, src=(0, 1, 3), cpml_width=1, cpml_f0=30.0,
                   rec=np.array([(0, 0, 5), (1, 1, 2)]), tune=False)
        tr = s.run(nt, wav)
        assert s.sync_status() == 0
        out.append((tr, s.read_field(0)[:12].clone()))
        s.close()
        del s
    assert out[0][1].abs().max() > 0
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])


def test_more_planes_than_32_bit_table_offsets_hold():
    """1 x 1 x (2^29 + 1000) nodes, source and receivers in the last planes:
    what a grid of 1000 planes gives at its end, where nothing from the other
    end arrives (4 planes a step)."""
    from paper_2404_04441_amd import Solver

    nt = 6
    wav = torch.from_numpy(ricker(nt, DT, 60.0, t0=2 * DT)).cuda()
    out = []
    for nz in (1000, (1 << 29) + 1000):
        print(f"case: 1 x 1 x {nz}", flush=True)
        rec = np.array([(0, 0, nz - 30 + k) for k in range(0, 30, 3)])
        s = Solver(torch.full((nz, 1, 1), 3000.0, device="cuda"), H, DT, src=(0, 0, nz - 9), rec=rec, tune=False)
        tr = s.run(nt, wav)
        assert s.sync_status() == 0
        out.append((tr, s.read_field(0)[-60:].clone()))
        s.close()
        del s
    assert out[0][1].abs().max() > 0
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
