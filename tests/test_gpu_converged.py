"""GPU tests of instances that have nothing to do: a state whose initial
residual is already below the tolerance takes no cycle, and the step returns it
unchanged, whatever the parity of the smoothing launches on the finest level
(their out-of-place copies), alone and beside instances that take cycles.
"""
import numpy as np
import pytest

from workloads import uniform_field

pytestmark = pytest.mark.gpu

# an odd number of out-of-place launches on the finest level a cycle: 2D tiles
# and strips, 3D bricks of one and of two steps a launch, the fused 3D step
CASES = [((128, 128), dict(nu1=3, nu2=2)), ((128, 128), dict(nu1=3, nu2=2, smoother=2)),
         ((128, 128), dict(nu1=2, nu2=3, precision=1)), ((48, 32, 64), dict(nu1=2, nu2=1)),
         ((48, 32, 64), dict(nu1=1, nu2=2)), ((16, 16, 16), dict(nu1=3, nu2=2)),
         ((16, 16, 16), dict(nu1=1, nu2=3)), ((32, 32, 32), dict(nu1=2, nu2=1, smoother=4)),
         ((48, 32, 64), dict(nu1=2, nu2=1, precision=1))]


@pytest.fixture(scope="module")
def chhs():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from paper_1611_02967_amd import chhs as binding
    return binding


def _state(fields):
    import torch
    phi = torch.from_numpy(np.concatenate([f.ravel() for f in fields])).to("cuda")
    return [phi, phi.clone(), torch.zeros_like(phi), torch.zeros_like(phi)]


def _solver(chhs, shapes, opts):
    return chhs.Solver([chhs.make_problem(s, 1.0 / s[-1], 0.05, 2.0, 5e-4) for s in shapes],
                       chhs.chhs_default_opts(**opts))


@pytest.mark.parametrize("shape,opts", CASES)
@pytest.mark.parametrize("use_graph", [1, 0])
def test_converged_state_comes_back_unchanged(chhs, shape, opts, use_graph):
    """phi = mu = p = 0 solves the step exactly; the context has stepped another
    state before, so that its workspace holds something else."""
    sv = _solver(chhs, [shape], dict(opts, use_graph=use_graph))
    sv.step(*_state([uniform_field(shape, 9500, mean=0.1, amp=0.3)]), 1)
    zero = _state([np.zeros(shape)])
    for _ in range(2):
        _, st = sv.step(*zero, 2)
        assert st[0]["total_vcycles"] == 0
        for v in zero:
            assert bool((v == 0.0).all())


@pytest.mark.parametrize("shape,opts", CASES)
def test_converged_instance_beside_an_active_one(chhs, shape, opts):
    sv = _solver(chhs, [shape, shape], opts)
    active = uniform_field(shape, 9501, mean=0.1, amp=0.3)
    n = active.size
    # the instance has been stepped from another state before
    sv.step(*_state([uniform_field(shape, 9502, mean=-0.1, amp=0.3), active]), 1)
    both = _state([np.zeros(shape), active])
    _, st = sv.step(*both, 1)
    assert st[0]["vcycles"] == 0 and st[1]["vcycles"] > 1
    for v in both:
        assert bool((v[:n] == 0.0).all())
    alone = _state([active])
    _, sa = _solver(chhs, [shape], opts).step(*alone, 1)
    assert sa[0]["vcycles"] == st[1]["vcycles"]
    for v, w in zip(both, alone):
        assert float((v[n:] - w).abs().max()) <= 1e-12
