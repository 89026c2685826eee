"""The symmetric adjoint products (FP32 and split BF16) at the edges of their shell blocks,
pairs of partners and stages, against the FP64 oracle gradient.

Tolerance: 1e-4 relative L2 over the grid, the gate of the other gradient tests.
"""
import numpy as np
import pytest

import fieldgen
import oracle as O

pytestmark = pytest.mark.gpu
_CACHE = {}


def _reference(N, order, nb, width, aliased, seed):
    key = (N, order, nb, width, aliased)
    if key not in _CACHE:
        delta = fieldgen.lognormal_field(N, seed).astype(np.float32)
        _CACHE[key] = delta, O.polyspectrum(delta.astype(np.float64), order, nb, width, return_fields=True,
                                            allow_aliasing=aliased)
    return _CACHE[key]


def _check(N, order, nb, width, precision, aliased=False, seed=61):
    import torch

    import paper_1904_11055_amd as ps
    delta, ref = _reference(N, order, nb, width, aliased, seed)
    g = np.random.default_rng(nb).standard_normal(len(ref["B"]))
    gref = O.gradient(delta.astype(np.float64), order, nb, width, g, result=ref, allow_aliasing=aliased)
    plan = ps.Plan(N, order, nb, width, precision=precision, flags=ps.ALLOW_ALIASING if aliased else 0, device="cuda:0")
    plan.shells(torch.from_numpy(delta)[None].to("cuda:0"))
    got = plan.backward(torch.from_numpy(g)[None].to("cuda:0")).cpu().numpy()[0]
    plan.close()
    assert np.linalg.norm(got - gref) < 1e-4 * np.linalg.norm(gref)


@pytest.mark.timeout(600)
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("nb", [9, 15, 16, 17, 32, 33, 47, 48, 49, 64])
def test_order3_shell_blocks(gpu, nb, precision):
    """Last blocks of 1, 15 and 16 shells, odd partner pairs and partial stages."""
    _check(32 if nb <= 42 else 64, 3, nb, 0.25, precision)


@pytest.mark.timeout(600)
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("nb", [40, 63])
def test_order3_aliased(gpu, nb, precision):
    """An aliased plan closes triplets outside the triangle bound: no weight block is skipped."""
    _check(32, 3, nb, 0.25, precision, aliased=True)


@pytest.mark.timeout(600)
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("nb", [9, 15, 16, 17, 24, 31])
def test_order4_shell_blocks(gpu, nb, precision):
    _check(32, 4, nb, 0.25, precision)


@pytest.mark.timeout(900)
@pytest.mark.parametrize("precision", [0, 1])
def test_order4_four_blocks(gpu, precision):
    """50 shells: all four shell blocks of the order-4 form, the last one with one pair."""
    _check(64, 4, 50, 0.25, precision)
