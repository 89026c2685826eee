"""Every raw sum of the order-3 and order-4 contractions against the FP64 oracle, each tuple by its own size.

Tolerance: the gate of the raw sums, |S - S_ref| relative to sum_x |prod_j d_{t_j}[x]|, at the
stated value (1e-5 FP32, 1e-4 splits) times order / 3.  Half of the sums are above 1e-2 of that
size and 98% above twice the gate, so that a missing or misplaced one shows whatever the size of
the others.
"""
import numpy as np
import pytest

import fieldgen
import oracle as O

pytestmark = pytest.mark.gpu
_CACHE = {}
TOL = {0: 1e-5, 1: 1e-4, 2: 1e-4}
SEEDS = (73, 74)      # the fields of the batch


def _reference(N, order, nb, width, aliased):
    key = (N, order, nb, width, aliased)
    if key not in _CACHE:
        _CACHE.clear()
        out = []
        for seed in SEEDS:
            delta = fieldgen.lognormal_field(N, seed).astype(np.float32)
            ref = O.polyspectrum(delta.astype(np.float64), order, nb, width, return_fields=True,
                                 allow_aliasing=aliased)
            size = O.product_sums(np.abs(ref["fields"]), ref["tuples"])
            out.append((delta, ref["tuples"], ref["sums"], size))
        _CACHE[key] = out
    return _CACHE[key]


def _check(N, order, nb, width, precision, aliased, all_shells):
    """A plan of nb shells against the tuples of the largest plan that it shares."""
    import torch

    import paper_1904_11055_amd as ps
    refs = _reference(N, order, all_shells, width, aliased)
    plan = ps.Plan(N, order, nb, width, batch=len(refs), precision=precision,
                   flags=ps.ALLOW_ALIASING if aliased else 0, device="cuda:0")
    plan.shells(torch.from_numpy(np.stack([r[0] for r in refs])).to("cuda:0"))
    S = plan.contract(raw=True)[1].cpu().numpy()
    got = plan.tuples
    plan.close()
    for b, (_, tuples, sums, size) in enumerate(refs):
        keep = tuples.max(axis=1) <= nb
        assert np.array_equal(got, tuples[keep])
        tol = TOL[precision] * order / 3
        assert np.mean(np.abs(sums[keep]) > 2 * tol * size[keep]) > 0.98
        assert np.max(np.abs(S[b] - sums[keep]) / size[keep]) < tol


@pytest.mark.timeout(600)
@pytest.mark.parametrize("nb", [9, 16, 24, 28, 29, 30, 31])
@pytest.mark.parametrize("precision", [2, 1, 0])
def test_order4(gpu, precision, nb):
    """Up to 28 pair blocks (29 shells) in one layout of the FP16 split, more in the other."""
    _check(32, 4, nb, 0.25, precision, False, 31)


@pytest.mark.timeout(600)
@pytest.mark.parametrize("nb", [24, 30, 41, 42])
def test_order4_aliased(gpu, nb):
    """Every tile of the pair products in use; 42 shells are 57 pair blocks."""
    _check(32, 4, nb, 0.25, 2, True, 42)


@pytest.mark.timeout(900)
@pytest.mark.parametrize("nb", [41, 48, 50])
def test_order4_many_blocks(gpu, nb):
    _check(64, 4, nb, 0.25, 2, False, 50)


@pytest.mark.timeout(900)
@pytest.mark.parametrize("precision,nb", [(2, n) for n in (7, 8, 9, 16, 17, 24, 33, 48, 49, 57, 63, 64)] +
                         [(p, n) for p in (0, 1) for n in (9, 16, 40, 64)])
def test_order3(gpu, precision, nb):
    """Shells that fill a product operand alone, share one from either end or leave it half empty."""
    _check(64, 3, nb, 0.25, precision, False, 64)


@pytest.mark.timeout(600)
@pytest.mark.parametrize("nb", [24, 48, 63])
def test_order3_aliased(gpu, nb):
    """The corner tiles included."""
    _check(32, 3, nb, 0.25, 2, True, 63)
