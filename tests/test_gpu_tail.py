"""GPU tests of the one-workgroup coarse tail at the sizes where its layout
changes: one wave, several waves, levels that share a wave, odd coarsest
extents, the last sizes whose pairs of cells each get an owner thread and the
first that do not.

One V-cycle agrees with the oracle's iterate by iterate to 1e-11 (some hundred
roundings of values of order one, amplified by at most 1 / (h^2 s) in p); a
mixed-precision step agrees with the oracle's to 1e-8, as both solve to 1e-10.
"""
import numpy as np
import pytest

from oracle import fas, scheme
from workloads import uniform_field

pytestmark = pytest.mark.gpu

SHAPES = [(4, 4), (14, 10), (12, 6), (8, 16), (16, 16), (28, 20), (24, 48), (32, 40), (64, 80),
          (4, 4, 4), (6, 10, 14), (8, 8, 12), (8, 12, 10), (16, 24, 20)]


@pytest.fixture(scope="module")
def chhs():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from paper_1611_02967_amd import chhs as binding
    return binding


def dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


def _inputs(shape, seed):
    prev = uniform_field(shape, seed, amp=0.6)
    cur = prev + uniform_field(shape, seed + 1, amp=0.1)
    return prev, cur, uniform_field(shape, seed + 2, amp=0.3), uniform_field(shape, seed + 3, amp=0.01)


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("variant", [dict(), dict(prolong=1), dict(order=1)],
                         ids=["plain", "bilinear", "first-order"])
def test_one_vcycle_matches_oracle(chhs, shape, variant):
    prm = scheme.Params(eps=0.05, gamma=2.0, s=1e-3, h=1.0 / shape[-1],
                        order=variant.get("order", 2))
    prev, cur, mu0, p0 = _inputs(shape, 8100)
    sv = chhs.Solver(chhs.make_problem(shape, prm.h, prm.eps, prm.gamma, prm.s),
                     chhs.chhs_default_opts(**variant))
    sv.setup_step(dev(prev), dev(cur), dev(mu0), dev(p0))
    sv.fas_vcycle()
    phi_star, f = scheme.step_rhs(prev, cur, prm)
    levels = fas.build_levels(phi_star, cur.copy(), f, prm.h)
    us = [None] * len(levels)
    us[0] = u = [cur.copy(), mu0.copy(), p0 - p0.mean()]
    fas.vcycle(levels, us, 0, prm,
               fas.Opts(prolong="bilinear" if variant.get("prolong") else "constant"))
    u[2] -= u[2].mean()
    for name, want in zip(("phi", "mu", "p"), u):
        got = sv.read_field(0, name).cpu().numpy()
        assert np.max(np.abs(got - want)) <= 1e-11, name


@pytest.mark.parametrize("shape", SHAPES)
def test_mixed_step_matches_oracle(chhs, shape):
    prm = scheme.Params(eps=0.05, gamma=2.0, s=1e-3, h=1.0 / shape[-1])
    prev, cur, mu0, p0 = _inputs(shape, 8200)
    sv = chhs.Solver(chhs.make_problem(shape, prm.h, prm.eps, prm.gamma, prm.s),
                     chhs.chhs_default_opts(precision=1))
    t = [dev(v) for v in (prev, cur, mu0, p0)]
    sv.step(*t, 1)
    ref = fas.solve_step(prev, cur, mu0, p0 - p0.mean(), prm, fas.Opts(tol=1e-10))
    assert np.max(np.abs(t[1].cpu().numpy() - ref.phi)) <= 1e-8
    assert np.max(np.abs(t[2].cpu().numpy() - ref.mu)) <= 1e-8


# every instance's finest level in the tail: the cycles of a step are one launch
@pytest.mark.parametrize("shapes", [[(16, 16)], [(32, 32), (4, 4), (14, 10)], [(8, 8, 8), (4, 4, 4)]],
                         ids=["16", "ragged", "3d"])
def test_steps_held_by_the_tail_match_cycle_launches_and_oracle(chhs, shapes):
    import torch
    prms = [scheme.Params(eps=0.1, gamma=2.0, s=1e-3, h=1.0 / sh[-1]) for sh in shapes]
    ins = [_inputs(sh, 8300 + 10 * i) for i, sh in enumerate(shapes)]
    probs = [chhs.make_problem(sh, q.h, q.eps, q.gamma, q.s) for sh, q in zip(shapes, prms)]

    def state():
        return [torch.cat([dev(v[k].reshape(-1)) for v in ins]) for k in range(4)]
    one, many = state(), state()
    _, a = chhs.Solver(probs, chhs.chhs_default_opts()).step(*one, 2)
    # a context that times its kernels launches every cycle
    _, b = chhs.Solver(probs, chhs.chhs_default_opts(timing=1)).step(*many, 2)
    for x, y in zip(one, many):
        assert torch.equal(x, y)
    assert [(s["vcycles"], s["total_vcycles"]) for s in a] == [(s["vcycles"], s["total_vcycles"])
                                                               for s in b]
    at = 0
    for sh, prm, (prev, cur, mu, p) in zip(shapes, prms, ins):
        for _ in range(2):
            r = fas.solve_step(prev, cur, mu, p - p.mean(), prm, fas.Opts(tol=1e-10))
            prev, cur, mu, p = cur, r.phi, r.mu, r.p
        got = one[1][at:at + cur.size].cpu().numpy().reshape(sh)
        assert np.max(np.abs(got - cur)) <= 1e-9
        at += cur.size


def test_step_held_by_the_tail_stops_at_max_vcycles(chhs):
    sh = (16, 16)
    sv = chhs.Solver(chhs.make_problem(sh, 1.0 / 16, 0.1, 2.0, 1e-3),
                     chhs.chhs_default_opts(max_vcycles=2))
    t = [dev(v) for v in _inputs(sh, 8400)]
    before = [v.clone() for v in t]
    rc, st = sv.step(*t, 1, check=False)
    assert rc == chhs.CHHS_E_NOCONV and st[0]["vcycles"] == 2 and st[0]["res_norm"] > 1e-10
    for x, y in zip(t, before):
        assert bool((x == y).all())


@pytest.mark.parametrize("nu", [(3, 2), (2, 3)])
@pytest.mark.parametrize("precision", [0, 1], ids=["fp64", "mixed"])
def test_odd_launches_on_a_level_leave_the_tails_of_other_instances_alone(chhs, nu, precision):
    """A level that some instances smooth by an odd number of out-of-place
    launches and others hold in their tail: every instance as alone, bit for bit."""
    import torch
    shapes = [(128, 128), (32, 32), (64, 64)]
    phi0 = [uniform_field(s, 9400 + i, mean=0.1, amp=0.05) for i, s in enumerate(shapes)]

    def run(idx):
        probs = [chhs.make_problem(shapes[i], 1.0 / shapes[i][-1], 0.05, 2.0, 5e-4) for i in idx]
        sv = chhs.Solver(probs, chhs.chhs_default_opts(nu1=nu[0], nu2=nu[1], precision=precision))
        t = torch.from_numpy(np.concatenate([phi0[i].ravel() for i in idx])).to("cuda")
        st = [t.clone(), t.clone(), torch.zeros_like(t), torch.zeros_like(t)]
        _, stats = sv.step(*st, 2)
        off = np.cumsum([0] + [phi0[i].size for i in idx])
        return [[v.cpu().numpy()[off[k]:off[k + 1]] for v in st] + [stats[k]["vcycles"]]
                for k in range(len(idx))]
    batch = run([0, 1, 2])
    for i in range(3):
        for a, b in zip(batch[i], run([i])[0]):
            assert np.array_equal(a, b), i
