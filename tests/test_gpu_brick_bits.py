"""GPU tests: smoothing in bricks has the bits of the per-color launches, and batches
on either side of the size up to which a finest level is in bricks agree."""
import numpy as np
import pytest

from workloads import uniform_field

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def chhs():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from paper_1611_02967_amd import chhs as binding
    return binding


@pytest.mark.parametrize("shape", [(16, 16, 16), (12, 20, 28), (24, 24, 24), (48, 32, 64), (40, 56, 24)])
@pytest.mark.parametrize("nu,prolong", [((2, 2), 0), ((1, 3), 0), ((2, 1), 0), ((3, 1), 1)])
def test_one_vcycle_has_the_bits_of_the_per_color_launches(chhs, shape, nu, prolong):
    """One V-cycle from the same level data (the setup has taken p's mean out):
    phi and mu bit for bit."""
    import torch
    state = [uniform_field(shape, 9700 + k, mean=0.1, amp=a) for k, a in enumerate((0.3, 0.3, 0.3, 0.01))]
    out = []
    for smoother in (3, 0):
        sv = chhs.Solver(chhs.make_problem(shape, 1.0 / shape[-1], 0.05, 2.0, 1e-3),
                         chhs.chhs_default_opts(nu1=nu[0], nu2=nu[1], prolong=prolong, smoother=smoother))
        sv.setup_step(*[torch.from_numpy(v).to("cuda") for v in state])
        sv.fas_vcycle()
        out.append([sv.read_field(0, n).cpu().numpy() for n in ("phi", "mu")])
    for a, b in zip(*out):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("precision,most", [(0, 12), (1, 16)], ids=["fp64", "mixed"])
def test_batches_about_the_largest_in_bricks(chhs, precision, most):
    """`most` grids of 32^3 have their finest level in bricks, one more smooth it
    per color: the same updates, sums over the grid in another order (1e-13)."""
    import torch
    phi0 = [torch.from_numpy(uniform_field((32, 32, 32), 9750 + i, mean=0.1, amp=0.1).ravel()) for i in range(3)]
    out = []
    for count in (most, most + 1):
        sv = chhs.Solver([chhs.make_problem((32, 32, 32), 1.0 / 32, 0.05, 2.0, 5e-4)] * count,
                         chhs.chhs_default_opts(precision=precision))
        phi = torch.cat([phi0[i % 3] for i in range(count)]).to("cuda")
        t = [phi, phi.clone(), torch.zeros_like(phi), torch.zeros_like(phi)]
        assert (sv.level_kernels()[0][1] == 1) == (count == most)      # steps per launch
        _, st = sv.step(*t, 1)
        out.append([v[:3 * 32 ** 3] for v in t] + [[s["vcycles"] for s in st[:3]]])
    assert out[0][4] == out[1][4]
    for a, b in zip(out[0][:4], out[1][:4]):
        assert float((a - b).abs().max()) <= 1e-13
