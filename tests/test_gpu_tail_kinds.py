"""GPU test: batches whose instances share the owner threads of their coarse tails
(equal extents, at the finest level or below it) beside others that do not.
"""
import numpy as np
import pytest

from workloads import uniform_field

pytestmark = pytest.mark.gpu

BATCHES = {"2d": [(16, 16), (32, 32), (16, 16), (14, 10), (64, 64), (32, 32), (40, 32), (128, 128), (14, 10)],
           "3d": [(8, 8, 8), (16, 16, 16), (8, 8, 8), (10, 10, 10), (4, 8, 8), (16, 16, 16)]}


@pytest.mark.parametrize("precision", [0, 1], ids=["fp64", "mixed"])
@pytest.mark.parametrize("name", list(BATCHES))
def test_instances_of_equal_tails_have_the_bits_of_their_single_runs(name, precision):
    import torch
    from paper_1611_02967_amd import chhs
    shapes = BATCHES[name]
    phi0 = [uniform_field(s, 9850 + i, mean=0.1, amp=0.2) for i, s in enumerate(shapes)]

    def run(idx):
        probs = [chhs.make_problem(shapes[i], 1.0 / shapes[i][-1], 0.05 + 0.01 * i, 1.0 + 0.2 * i, 5e-4)
                 for i in idx]
        sv = chhs.Solver(probs, chhs.chhs_default_opts(precision=precision))
        phi = torch.from_numpy(np.concatenate([phi0[i].ravel() for i in idx])).to("cuda")
        t = [phi, phi.clone(), torch.zeros_like(phi), torch.zeros_like(phi)]
        _, st = sv.step(*t, 2)
        off = np.cumsum([0] + [phi0[i].size for i in idx])
        return [[v[off[k]:off[k + 1]].cpu().numpy() for v in t] + [st[k]["vcycles"]] for k in range(len(idx))]
    batch = run(range(len(shapes)))
    for i in range(len(shapes)):
        for a, b in zip(batch[i], run([i])[0]):
            assert np.array_equal(a, b), shapes[i]
