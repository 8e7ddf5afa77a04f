"""GPU tests of FP64 2D batches that hold large instances (finest level in
row-streaming strips) beside small ones (in tiles): every instance is smoothed
as it is alone.
"""
import numpy as np
import pytest

from workloads import uniform_field

pytestmark = pytest.mark.gpu

SHAPES = [(64, 64), (2048, 1536), (96, 160), (16, 16), (512, 256)]      # 2048 x 1536 = 3 2^20 cells


@pytest.fixture(scope="module")
def chhs():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from paper_1611_02967_amd import chhs as binding
    return binding


def _run(chhs, idx, steps=2, **opts):
    import torch
    probs = [chhs.make_problem(SHAPES[i], 1.0 / SHAPES[i][-1], 0.02, 2.0, 1e-4) for i in idx]
    sv = chhs.Solver(probs, chhs.chhs_default_opts(**opts))
    phi = torch.from_numpy(np.concatenate([uniform_field(SHAPES[i], 9000 + i, mean=0.1, amp=0.1).ravel()
                                           for i in idx])).to("cuda")
    t = [phi, phi.clone(), torch.zeros_like(phi), torch.zeros_like(phi)]
    _, st = sv.step(*t, steps)
    off = np.cumsum([0] + [int(np.prod(SHAPES[i])) for i in idx])
    return sv, [[v[off[k]:off[k + 1]].cpu().numpy() for v in t] + [st[k]["res_norm"], st[k]["vcycles"]]
                for k in range(len(idx))]


@pytest.mark.parametrize("nu", [(2, 2), (3, 2)])
@pytest.mark.parametrize("idx", [[0, 1], [4, 2, 1, 3]])
def test_every_instance_has_the_bits_of_its_single_run(chhs, idx, nu):
    sv, batch = _run(chhs, idx, nu1=nu[0], nu2=nu[1])
    assert sv.level_kernels()[0][0] == "strips"
    for k, i in enumerate(idx):
        alone = _run(chhs, [i], nu1=nu[0], nu2=nu[1])[1][0]
        for a, b in zip(batch[k], alone):
            assert np.array_equal(a, b), i


def test_tuned_batch_takes_one_kernel_for_all(chhs):
    """The autotuner cuts the level's tables anew: the same steps to the tolerance."""
    want = _run(chhs, [0, 1, 2], 1)[1]
    got = _run(chhs, [0, 1, 2], 1, autotune=1)[1]
    for a, b in zip(got, want):
        assert a[5] == b[5]
        assert np.max(np.abs(a[1] - b[1])) <= 1e-10
