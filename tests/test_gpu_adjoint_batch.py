"""Batched gradients: every entry of a batch has its own fields, weights and repeated-shell weights.

Tolerance: 1e-4 relative L2 over the grid, the gate of the other gradient tests.
"""
import numpy as np
import pytest

import fieldgen
import oracle as O

pytestmark = pytest.mark.gpu
_CACHE = {}
SEEDS = (31, 32, 33)


def _reference(N, order, nb, width):
    key = (N, order, nb, width)
    if key not in _CACHE:
        _CACHE.clear()
        out = []
        for seed in SEEDS:
            delta = fieldgen.lognormal_field(N, seed).astype(np.float32)
            ref = O.polyspectrum(delta.astype(np.float64), order, nb, width, return_fields=True)
            g = np.random.default_rng(seed).standard_normal(len(ref["B"]))
            out.append((delta, ref, g))
        _CACHE[key] = out
    return _CACHE[key]


@pytest.mark.timeout(600)
@pytest.mark.parametrize("precision", [0, 1, 2])
@pytest.mark.parametrize("half", [False, True])
@pytest.mark.parametrize("order,nb", [(3, 12), (3, 40), (4, 12), (4, 17), (4, 31)])
def test_gradient_of_a_batch(gpu, order, nb, precision, half):
    import torch

    import paper_1904_11055_amd as ps
    N, width = 32, 0.25
    refs = _reference(N, order, nb, width)
    x = np.stack([r[0] for r in refs])
    if half:
        x = np.fft.rfftn(x.astype(np.float64), axes=(1, 2, 3)).astype(np.complex64)
    plan = ps.Plan(N, order, nb, width, batch=len(refs), precision=precision,
                   flags=ps.INPUT_HALF_SPECTRUM if half else 0, device="cuda:0")
    plan.shells(torch.from_numpy(x).to("cuda:0"))
    got = plan.backward(torch.from_numpy(np.stack([r[2] for r in refs])).to("cuda:0")).cpu().numpy()
    plan.close()
    for b, (delta, ref, g) in enumerate(refs):
        if half:
            want = O.gradient_half_spectrum(N, order, nb, width, ref["tuples"], ref["counts"], ref["fields"], g)
        else:
            want = O.gradient(delta.astype(np.float64), order, nb, width, g, result=ref)
        assert np.linalg.norm(got[b] - want) < 1e-4 * np.linalg.norm(want), b
