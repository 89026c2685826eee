"""The order-3 contraction by aligned products at the edges of its shell blocks: shells that fill a product
operand alone, share one from either end, or leave it half empty, against the FP64 oracle.

Tolerance: 1e-4 relative L2 over the tuples, the gate of the split-precision contraction.
"""
import numpy as np
import pytest

import fieldgen
import oracle as O

pytestmark = pytest.mark.gpu
_CACHE = {}


def _reference(N, nb, width, aliased):
    key = (N, nb, width, aliased)
    if key not in _CACHE:
        delta = fieldgen.lognormal_field(N, 71).astype(np.float32)
        _CACHE[key] = delta, O.polyspectrum(delta.astype(np.float64), 3, nb, width, allow_aliasing=aliased)
    return _CACHE[key]


def _check(N, nb, width, aliased, all_shells, precision=2):
    """A plan of nb shells against the tuples of the largest plan that it shares."""
    import torch

    import paper_1904_11055_amd as ps
    delta, ref = _reference(N, all_shells, width, aliased)
    keep = ref["tuples"].max(axis=1) <= nb
    plan = ps.Plan(N, 3, nb, width, precision=precision, flags=ps.ALLOW_ALIASING if aliased else 0, device="cuda:0")
    plan.shells(torch.from_numpy(delta)[None].to("cuda:0"))
    B, S = (v.cpu().numpy()[0] for v in plan.contract(raw=True))
    assert np.array_equal(plan.tuples, ref["tuples"][keep])
    plan.close()
    want = ref["B"][keep]
    assert np.linalg.norm(B - want) < 1e-4 * np.linalg.norm(want)
    # every tuple against the magnitude of its own block of shells, so that one misplaced
    # entry among thousands shows
    scale = np.abs(want).max() * 1e-4 + 2e-2 * np.abs(want)
    assert np.all(np.abs(B - want) < scale)


@pytest.mark.timeout(600)
@pytest.mark.parametrize("nb", [7, 8, 9, 15, 16, 17, 23, 24, 25, 31, 32, 33, 40, 41, 47, 48, 49, 55, 56, 57, 63, 64])
def test_shell_blocks(gpu, nb):
    _check(64, nb, 0.25, False, 64)


@pytest.mark.timeout(600)
@pytest.mark.parametrize("nb", [24, 48, 63])
def test_aliased(gpu, nb):
    """Aliased: every tuple closes, the corner tiles included."""
    _check(32, nb, 0.25, True, 63)


@pytest.mark.timeout(600)
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("nb", [9, 16, 40, 48, 49, 63, 64])
def test_other_precisions(gpu, nb, precision):
    """FP32 and BF16 on the plans that take the aligned products (one block), and on others."""
    _check(64, nb, 0.25, False, 64, precision)
