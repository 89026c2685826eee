"""The order-4 split-FP16 contraction at the edges of its pair blocks, slots and groups, against the FP64 oracle.

Tolerance: 1e-4 relative L2 over the tuples, the gate of the split-precision contraction.
"""
import numpy as np
import pytest

import fieldgen
import oracle as O

pytestmark = pytest.mark.gpu
_CACHE = {}
N = 32


def _reference(nb, width, aliased):
    key = (nb, width, aliased)
    if key not in _CACHE:
        delta = fieldgen.lognormal_field(N, 73).astype(np.float32)
        _CACHE[key] = delta, O.polyspectrum(delta.astype(np.float64), 4, nb, width, allow_aliasing=aliased)
    return _CACHE[key]


def _check(nb, width, aliased, all_shells):
    """A plan of nb shells against the tuples of the largest plan that it shares."""
    import torch

    import paper_1904_11055_amd as ps
    delta, ref = _reference(all_shells, width, aliased)
    keep = ref["tuples"].max(axis=1) <= nb
    plan = ps.Plan(N, 4, nb, width, precision=ps.SPLIT_FP16, flags=ps.ALLOW_ALIASING if aliased else 0,
                   device="cuda:0")
    plan.shells(torch.from_numpy(delta)[None].to("cuda:0"))
    B = plan.contract(raw=True)[0].cpu().numpy()[0]
    assert np.array_equal(plan.tuples, ref["tuples"][keep])
    plan.close()
    want = ref["B"][keep]
    assert np.linalg.norm(B - want) < 1e-4 * np.linalg.norm(want)
    # every tuple against its own size too, so that one misplaced entry among thousands shows
    assert np.all(np.abs(B - want) < np.abs(want).max() * 1e-4 + 2e-2 * np.abs(want))


@pytest.mark.timeout(300)
@pytest.mark.parametrize("nb", [8, 9, 11, 15, 16, 17, 20, 22, 24, 28, 29, 30, 31])
def test_pair_blocks(gpu, nb):
    """Up to 28 pair blocks (29 shells) in one layout, more in the other."""
    _check(nb, 0.25, False, 31)


@pytest.mark.timeout(300)
@pytest.mark.parametrize("nb", [41, 42, 48, 63])
def test_many_blocks(gpu, nb):
    """More pair blocks than a group may hold (56, at 42 shells)."""
    _check(nb, 0.125, False, 63)


@pytest.mark.timeout(300)
@pytest.mark.parametrize("nb", [24, 30, 42])
def test_aliased(gpu, nb):
    """Aliased: every tile of the pair products in use."""
    _check(nb, 0.25, True, 42)
