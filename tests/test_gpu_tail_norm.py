"""GPU test: the residual norm that the coarse tail forms of a finest level it
holds, at sizes whose pairs of cells do not fill its waves (14 x 10 leaves six in
the second wave, 4 x 4 shares one wave with the coarser levels).
"""
import pytest

from workloads import uniform_field

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def chhs():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from paper_1611_02967_amd import chhs as binding
    return binding


@pytest.mark.parametrize("shape", [(4, 4), (14, 10), (12, 6), (16, 16), (28, 20), (4, 4, 4), (6, 10, 14)])
def test_norm_of_a_finest_level_held_by_the_tail(chhs, shape):
    """After each of three V-cycles, against the per-cell residual kernel on the
    iterate they left: some hundred terms summed in another order, 1e-12."""
    import torch
    sv = chhs.Solver(chhs.make_problem(shape, 1.0 / shape[-1], 0.1, 2.0, 1e-3), chhs.chhs_default_opts())
    sv.setup_step(*[torch.from_numpy(uniform_field(shape, 9800 + k, amp=0.3)).to("cuda") for k in range(4)])
    for _ in range(3):
        got = sv.fas_vcycle()[0]
        want = sv.residual_norms()[0][3]
        assert abs(got - want) <= 1e-12 * (1.0 + want)
        assert abs(float(sv.read_field(0, "p").mean())) <= 1e-15
