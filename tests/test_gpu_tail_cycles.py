"""GPU test: the cycles of a step that run in one launch (grids held by the coarse
tail) against cycles launched one by one.
"""
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


# at most 128 cycles a launch: the last one, one beyond, several launches
@pytest.mark.parametrize("cycles", [1, 2, 5, 127, 128, 129, 300])
def test_cycle_limit(chhs, cycles):
    """A tolerance below rounding is never met: every instance takes max_vcycles
    cycles, with the norms of a context that launches every cycle by itself (timed
    contexts do), bit for bit; a converged instance stays as it is."""
    import torch
    shapes = [(16, 16), (4, 4), (14, 10)]
    probs = [chhs.make_problem(s, 1.0 / s[-1], 0.1, 2.0, 1e-3) for s in shapes]
    phi = torch.from_numpy(np.concatenate([uniform_field(s, 9900 + i, amp=0.5).ravel() * (i != 1)
                                           for i, s in enumerate(shapes)])).to("cuda")
    runs = []
    for timing in (0, 1):
        sv = chhs.Solver(probs, chhs.chhs_default_opts(max_vcycles=cycles, tol=1e-18, timing=timing))
        t = [phi.clone(), phi.clone(), torch.zeros_like(phi), torch.zeros_like(phi)]
        rc, st = sv.step(*t, 1, check=False)
        assert rc == chhs.CHHS_E_NOCONV
        sol = torch.empty_like(phi)
        sv.get_solution(phi=sol)
        runs.append([[(s["vcycles"], s["status"], s["res_norm"]) for s in st], sol])
    assert [r[0] for r in runs[0][0]] == [cycles, 0, cycles]
    assert runs[0][0] == runs[1][0]
    assert torch.equal(runs[0][1], runs[1][1])
