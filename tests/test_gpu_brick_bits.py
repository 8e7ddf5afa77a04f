"""GPU test: FP64 smoothing in bricks has the bits of the per-color launches."""
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
