"""GPU test: the kernels reported for 3D levels are those the cycle launches."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,opts,want", [
    # bricks of 8 x 4 x 4 cells, two steps a launch up to 256 of them
    ((16, 16, 16), {}, [("per-cell", 2, 32)]),
    ((48, 32, 64), {}, [("per-cell", 1, 768), ("per-cell", 2, 96)]),
    ((128, 128, 128), {}, [("per-cell", 256, 4096), ("per-cell", 1, 2048), ("per-cell", 2, 256)]),
    ((32, 32, 32), dict(smoother=3), [("per-cell", 256, 64), ("per-cell", 256, 8)])])
def test_3d_levels_report_their_launches(shape, opts, want):
    from paper_1611_02967_amd import chhs
    sv = chhs.Solver(chhs.make_problem(shape, 1.0 / shape[-1], 0.05, 2.0, 1e-3),
                     chhs.chhs_default_opts(**opts))
    assert sv.level_kernels()[:len(want)] == want
