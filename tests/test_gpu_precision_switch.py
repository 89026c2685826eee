"""A plan switched to another precision gives, bit for bit, the sums of a plan made in it."""
import itertools

import numpy as np
import pytest

import fieldgen

pytestmark = pytest.mark.gpu


@pytest.mark.timeout(300)
@pytest.mark.parametrize("order,nb", [(3, 14), (3, 30), (4, 12), (4, 31), (5, 9), (6, 8), (6, 12)])
def test_sums_of_a_switched_plan(gpu, order, nb):
    """Order 4 with 31 shells has 31 pair blocks, more than one group of the narrow layout holds; order 6
    has tile groups of its own for FP32."""
    import torch

    import paper_1904_11055_amd as ps
    N, width = 64, 0.25
    x = torch.from_numpy(fieldgen.lognormal_field(N, 17).astype(np.float32))[None].to("cuda:0")
    made = {}
    for precision in (0, 1, 2):
        plan = ps.Plan(N, order, nb, width, precision=precision, device="cuda:0")
        plan.shells(x)
        made[precision] = plan, plan.contract(raw=True)[1].cpu().numpy()
    for first, then in itertools.permutations((0, 1, 2), 2):
        plan = made[first][0]
        plan.precision = then
        assert np.array_equal(plan.contract(raw=True)[1].cpu().numpy(), made[then][1]), (first, then)
        plan.precision = first
        assert np.array_equal(plan.contract(raw=True)[1].cpu().numpy(), made[first][1]), first
    for plan, _ in made.values():
        plan.close()
