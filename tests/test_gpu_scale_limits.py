"""Half storage on both sides of the difference of scales up to which a step
takes its factors in: the oracle's bound holds at each, and levels of sizes as
far apart as a float64 difference leaves them cost no more than equal ones."""
import time

import pytest

import test_gpu_storage_scales as scales
from synth import COURANT

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("apart", [38, 42, 58, 62])
@pytest.mark.parametrize("large", ["A", "V"])
def test_one_step_around_the_limits(apart, large):
    a, v = (1.0, 2.0 ** -apart) if large == "A" else (2.0 ** -apart, 1.0)
    scales.test_one_step_at_any_pair_of_scales("f16", a, v)


def test_a_float64_residue_is_no_slow_step():
    """V of 2^-53 of A: four steps take less than twice those from V of A's size
    (with the first one node by node, 4.7 times)."""
    from paper_2404_04441_amd import Solver

    shape = (256, 256, 256)
    s = Solver(torch.full(shape, 3000.0, device="cuda"), 10.0, COURANT * 10.0 / 4500.0, storage="f16", tune=False)
    a, v = (torch.randn(shape, device="cuda") for _ in range(2))
    took = {}
    for size in (1.0, 2.0 ** -53):
        best = 1e9
        for _ in range(5):
            s.write_field(0, a)
            s.write_field(2, v * size)
            torch.cuda.synchronize()
            t = time.perf_counter()
            s.step(4)
            torch.cuda.synchronize()
            best = min(best, time.perf_counter() - t)
        took[size] = best
    s.close()
    print(f"case: {took}", flush=True)
    assert took[2.0 ** -53] < 2 * took[1.0]
