"""Grids whose rows are padded inside the workspace: every entry point that
moves data between the caller's arrays and the fields, bit for bit against a
context with unpadded rows (an explicit one-node-per-lane shape)."""
import numpy as np
import pytest

from synth import COURANT, ricker, smooth_random

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _case(nx, rec_kind, nt=30):
    shape = (13, 17, nx)
    vel = smooth_random(shape, seed=81)
    dt = COURANT * 10.0 / 4500.0
    wav = ricker(nt, dt, 50.0)
    if rec_kind == "box":  # to the last column
        rec = np.array([(x, y, 4) for y in range(17) for x in range(nx)], dtype=np.int32)
    else:
        gen = np.random.default_rng(3)
        rec = np.stack([gen.integers(0, n, 40) for n in (nx, 17, 13)], 1).astype(np.int32)
        rec[0] = (nx - 1, 16, 12)
    return shape, vel, dt, nt, wav, rec


def _solver(vel, dt, rec, nx, **kw):
    from paper_2404_04441_amd import Solver

    return Solver(torch.from_numpy(vel).cuda(), 10.0, dt, src=(nx - 3, 8, 6), rec=rec, sponge_width=4,
                  sponge_alpha=0.05, **kw)


@pytest.mark.parametrize("nx", [33, 34, 71, 131, 301])
@pytest.mark.parametrize("rec_kind", ["box", "list"])
@pytest.mark.parametrize("storage,bits", [("f32", 32), ("f16", 32), ("bf16", 16)])
def test_padded_rows_are_bitwise_the_unpadded_ones(nx, rec_kind, storage, bits):
    shape, vel, dt, nt, wav, rec = _case(nx, rec_kind)
    w = torch.from_numpy(wav).cuda()
    print(f"case: nx {nx} {rec_kind} {storage} m{bits}", flush=True)
    gen = np.random.default_rng(9)
    fields = [torch.from_numpy((k * gen.standard_normal(shape)).astype(np.float32)).cuda() for k in (1.0, 0.05)]
    outs = []
    for kw in (dict(variant=7), dict(tune=False), dict(tune=True)):
        s = _solver(vel, dt, rec, nx, storage=storage, model_bits=bits, **kw)
        out = [s.run(nt, w), s.read_field(0), s.read_field(1)]
        snap = s.save_state()
        s.reset()
        s.write_field(0, fields[0])
        s.write_field(1 if storage == "f32" else 2, fields[1])
        out += [s.read_field(0), s.step(5, w)[:5], s.read_field(0), s.read_field(1)]
        s.load_state(snap)
        out += [s.read_field(0)]
        outs.append(([t.cpu().numpy() for t in out], snap, s))
    for got, snap, s in outs[1:]:
        assert not s.sync_status()
        for a, b in zip(got, outs[0][0]):
            assert np.array_equal(a, b)
        # a snapshot of unpadded rows resumes on padded ones
        s.load_state(outs[0][1])
        assert np.array_equal(s.read_field(0).cpu().numpy(), got[1])
    for _, _, s in outs:
        s.close()


@pytest.mark.parametrize("rec_kind", ["box", "list"])
def test_padded_gradient_and_tiling(rec_kind):
    nx = 71
    shape, vel, dt, nt, wav, rec = _case(nx, rec_kind)
    gen = np.random.default_rng(4)
    resid = torch.from_numpy(gen.standard_normal((nt, len(rec))).astype(np.float32)).cuda()
    w = torch.from_numpy(wav).cuda()
    grads = []
    for kw in (dict(variant=7), dict(tune=False), dict(tune=True)):
        s = _solver(vel, dt, rec, nx, adjoint=True, nt_max=nt, **kw)
        grads.append(s.adjoint(nt, w, resid).cpu().numpy())
        tiling = s.tiling()
        s.close()
        s = _solver(vel, dt, rec, nx, adjoint=True, nt_max=nt, tune=False, **tiling)
        assert s.tiling() == tiling
        s.close()
    assert np.abs(grads[0]).max() > 0
    assert np.array_equal(grads[1], grads[0]) and np.array_equal(grads[2], grads[0])


@pytest.mark.parametrize("storage", ["f32", "f16"])
def test_workspace_for_unpadded_rows_is_enough(storage):
    """A workspace of the unpadded size (an explicit one-node shape's) takes
    the library's choice of shape too, with the same bits."""
    import ctypes

    from paper_2404_04441_amd import _lib as L

    nx = 71
    shape, vel, dt, nt, wav, rec = _case(nx, "list")
    w = torch.from_numpy(wav).cuda()
    ref = _solver(vel, dt, rec, nx, storage=storage, variant=7)
    auto = _solver(vel, dt, rec, nx, storage=storage, tune=False)
    assert ref.workspace_bytes < auto.workspace_bytes
    want = [ref.run(nt, w).cpu(), ref.read_field(0).cpu(), ref.read_field(1).cpu()]
    p, v = auto._params, torch.from_numpy(vel).cuda()
    L.lib().wave_destroy(auto._h)
    auto._h = ctypes.c_void_p()
    assert L.lib().wave_create(ctypes.byref(p), v.data_ptr(), auto._ws_ptr, ref.workspace_bytes - 256,
                               auto.stream.cuda_stream, ctypes.byref(auto._h)) == L.WAVE_ENOSPC
    L.check(L.lib().wave_create(ctypes.byref(p), v.data_ptr(), auto._ws_ptr, ref.workspace_bytes,
                                auto.stream.cuda_stream, ctypes.byref(auto._h)), "wave_create")
    got = [auto.run(nt, w).cpu(), auto.read_field(0).cpu(), auto.read_field(1).cpu()]
    for a, b in zip(got, want):
        assert torch.equal(a, b)
    auto.close()
    ref.close()
