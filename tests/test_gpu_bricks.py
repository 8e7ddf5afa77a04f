"""GPU tests of the 3D smoothing in bricks: the same bits as the per-color
launches (opts.smoother = 3, which smooth, restrict, prolong and form right-hand
sides cell by cell), and the oracle's V-cycle.
"""
import numpy as np
import pytest

from oracle import fas, scheme
from workloads import uniform_field

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def chhs():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from paper_1611_02967_amd import chhs as binding
    return binding


def dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


def host(t):
    return t.detach().cpu().numpy()


def _vcycle(chhs, shape, prm, state, **opts):
    prob = chhs.make_problem(shape, prm.h, prm.eps, prm.gamma, prm.s)
    sv = chhs.Solver(prob, chhs.chhs_default_opts(**opts))
    sv.setup_step(*[dev(a) for a in state])
    res = sv.fas_vcycle()[0]
    return res, [host(sv.read_field(0, n)) for n in ("phi", "mu", "p")]


# (nz, ny, nx): one level above the tail and several, one and two steps a launch
# on the finest level, bricks cut by the grid in x, y and z
SHAPES = [(16, 16, 16), (12, 20, 28), (16, 24, 64), (24, 24, 24), (20, 12, 28), (48, 32, 64),
          (40, 56, 24)]


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("nu,prolong", [((2, 2), 0), ((1, 3), 0), ((3, 1), 1)])
def test_one_vcycle_in_bricks(chhs, shape, nu, prolong):
    """One V-cycle: phi and mu have the bits of the per-color launches; p and the
    norm differ by the order of their sums over the grid (p's mean is subtracted
    as p loads): 1e-13; the oracle to 1e-11."""
    prm = scheme.Params(eps=0.05, gamma=2.0, s=1e-3, h=1.0 / shape[-1])
    prev = uniform_field(shape, 9300, mean=0.1, amp=0.3)
    cur = prev + uniform_field(shape, 9301, amp=0.05)
    state = (prev, cur, uniform_field(shape, 9302, amp=0.3), uniform_field(shape, 9303, amp=0.01))
    kw = dict(nu1=nu[0], nu2=nu[1], prolong=prolong)
    want = _vcycle(chhs, shape, prm, state, smoother=3, **kw)
    got = _vcycle(chhs, shape, prm, state, **kw)
    phi_star, f = scheme.step_rhs(prev, cur, prm)
    levels = fas.build_levels(phi_star, cur.copy(), f, prm.h)
    u = [cur.copy(), state[2].copy(), state[3] - state[3].mean()]
    us = [u] + [None] * (len(levels) - 1)
    fas.vcycle(levels, us, 0, prm, fas.Opts(nu1=nu[0], nu2=nu[1],
                                           prolong="bilinear" if prolong else "constant"))
    u[2] -= u[2].mean()
    for k in range(3):
        scale = max(1.0, np.max(np.abs(u[k])))
        assert np.max(np.abs(got[1][k] - want[1][k])) <= 1e-13 * scale, k
        assert np.max(np.abs(got[1][k] - u[k])) <= 1e-11 * scale, k
    assert abs(got[0] - want[0]) <= 1e-13 * want[0]


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("nu,inner", [((2, 2), 1), ((1, 3), 2)])
def test_one_correction_in_bricks_has_the_bits_of_the_per_color_launches(chhs, shape, nu, inner):
    """Mixed precision, one refinement step: u + e with e from FP32 cycles."""
    prm = scheme.Params(eps=0.05, gamma=2.0, s=1e-3, h=1.0 / shape[-1])
    prev = uniform_field(shape, 9310, mean=0.1, amp=0.3)
    cur = prev + uniform_field(shape, 9311, amp=0.05)
    state = (prev, cur, uniform_field(shape, 9312, amp=0.3), uniform_field(shape, 9313, amp=0.01))
    kw = dict(nu1=nu[0], nu2=nu[1], precision=1, inner_cycles=inner)
    want = _vcycle(chhs, shape, prm, state, smoother=3, **kw)
    got = _vcycle(chhs, shape, prm, state, **kw)
    for k in range(2):
        assert np.array_equal(got[1][k], want[1][k]), k


def test_batch_with_bricks_of_one_and_two_steps_gives_the_single_runs_bits(chhs):
    """A batch whose levels take one step a launch where an instance alone takes
    two: every instance's steps keep the bits of its single run."""
    shapes = [(24, 24, 24), (48, 32, 64), (16, 24, 40)]
    phi0 = [uniform_field(s, 9320 + i, mean=0.1, amp=0.1) for i, s in enumerate(shapes)]

    def run(idx):
        probs = [chhs.make_problem(shapes[i], 1.0 / shapes[i][-1], 0.05, 2.0, 5e-4) for i in idx]
        sv = chhs.Solver(probs, chhs.chhs_default_opts())
        flat = np.concatenate([phi0[i].ravel() for i in idx])
        st = [dev(flat), dev(flat), dev(np.zeros(flat.size)), dev(np.zeros(flat.size))]
        _, stats = sv.step(*st, 2)
        off = np.cumsum([0] + [phi0[i].size for i in idx])
        return [([host(t)[off[k]:off[k + 1]] for t in st], stats[k]["vcycles"])
                for k in range(len(idx))]
    batch = run([0, 1, 2])
    for i in range(3):
        single = run([i])[0]
        assert batch[i][1] == single[1]
        for a, b in zip(batch[i][0], single[0]):
            assert np.array_equal(a, b), i
