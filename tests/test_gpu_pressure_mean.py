"""GPU tests of the pressure's free constant: a step does not depend on the mean
of the initial p, and the level's p that a program reads between calls is the
one of mean zero, on every smoothing path.
"""
import numpy as np
import pytest

from workloads import uniform_field

pytestmark = pytest.mark.gpu

# finest level in the tail (either kernel), tiles, bricks, per color, the fused
# 3D step, the first-order scheme, cycles without pre-smoothing
CASES = [((16, 16), {}), ((32, 32), {}), ((40, 32), {}), ((64, 64), {}), ((8, 8, 8), {}),
         ((10, 10, 10), {}), ((32, 32, 32), {}), ((32, 32, 32), dict(smoother=3)),
         ((32, 32, 32), dict(smoother=4)), ((80, 80, 80), {}), ((16, 16), dict(order=1)),
         ((64, 64), dict(order=1)), ((16, 16, 16), dict(order=1)), ((64, 64), dict(nu1=0, nu2=3)),
         ((16, 16, 16), dict(nu1=0, nu2=3))]


@pytest.fixture(scope="module")
def chhs():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from paper_1611_02967_amd import chhs as binding
    return binding


def _step(chhs, shape, opts, mean, nsteps=2):
    import torch
    sv = chhs.Solver(chhs.make_problem(shape, 1.0 / shape[-1], 0.05, 2.0, 1e-3),
                     chhs.chhs_default_opts(**opts))
    phi = torch.from_numpy(uniform_field(shape, 9600, mean=0.1, amp=0.3)).to("cuda")
    t = [phi, phi.clone(), torch.zeros_like(phi), torch.full_like(phi, mean)]
    _, st = sv.step(*t, nsteps)
    return sv, t, st[0]


@pytest.mark.parametrize("shape,opts", CASES)
@pytest.mark.parametrize("timing", [0, 1])
def test_step_from_a_pressure_with_a_large_mean(chhs, shape, opts, timing):
    """p0 = 1e6 against p0 = 0: p enters through differences alone, which are
    zero for both, so the steps agree to rounding (1e-12), as they can only if
    the mean is taken out before the first cycle (p's rounding at 1e6 is 1e-10)."""
    _, want, a = _step(chhs, shape, dict(opts, timing=timing), 0.0)
    _, got, b = _step(chhs, shape, dict(opts, timing=timing), 1e6)
    assert a["total_vcycles"] == b["total_vcycles"]
    for x, y in zip(got, want):
        assert float((x - y).abs().max()) <= 1e-12


@pytest.mark.parametrize("shape,opts", CASES)
def test_level_pressure_after_a_step_has_mean_zero(chhs, shape, opts):
    import torch
    sv, t, _ = _step(chhs, shape, opts, 0.0, 1)
    p = sv.read_field(0, "p")
    assert abs(float(p.mean())) <= 1e-14
    assert float((p - t[3]).abs().max()) <= 1e-15
    sol = torch.empty_like(p)
    sv.get_solution(p=sol)
    assert float((sol - t[3]).abs().max()) <= 1e-15


@pytest.mark.parametrize("shape", [(64, 64), (32, 32, 32)])
def test_solution_holds_the_pressure_written_to_the_level(chhs, shape):
    """Contexts whose cycles leave p's mean alone: a p written to the level comes
    back as it is, also after the residual norms were asked for."""
    import torch
    opts = dict(order=1) if len(shape) == 2 else dict(smoother=3)
    sv, t, _ = _step(chhs, shape, opts, 0.0, 1)
    p = t[3] + 0.25
    sv.write_field(0, "p", p)
    sv.residual_norms()
    sol = torch.empty_like(p)
    sv.get_solution(p=sol)
    assert bool((sol == p).all())
    assert bool((sv.read_field(0, "p") == p).all())
