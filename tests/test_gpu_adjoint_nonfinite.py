"""A non-finite dL/dB of one tuple stays with the shells of that tuple.

The gradient of a plan with half-spectrum input separates the shells: a mode belongs to one
shell.  A NaN weight makes the fields of its tuple's shells NaN, and those of the shells that
share a complex row transform with them (shells 2 i - 1 and 2 i); every other shell's part is
bit for bit that of a zero weight.
"""
import numpy as np
import pytest

import fieldgen

pytestmark = pytest.mark.gpu


def _shells(N, width):
    """Shell (1-based, real-valued edges) of every mode of the half spectrum."""
    k = np.fft.fftfreq(N, 1.0 / N)
    c = np.arange(N // 2 + 1)
    q = np.sqrt(k[:, None, None] ** 2 + k[None, :, None] ** 2 + c[None, None, :] ** 2)
    return np.floor(q / width + 0.5).astype(int)


@pytest.mark.timeout(300)
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("order,nb,tuple_", [(3, 15, (6, 14, 15)), (3, 27, (6, 14, 18)), (3, 27, (11, 11, 11)),
                                             (3, 44, (13, 21, 34)), (3, 60, (12, 40, 50)),
                                             (4, 14, (4, 6, 8, 9)), (4, 20, (4, 9, 13, 18)), (4, 20, (11, 18, 19, 20)),
                                             (4, 40, (6, 15, 28, 36)), (4, 52, (14, 20, 39, 50))])
def test_nan_weight_stays_with_its_shells(gpu, order, nb, tuple_, precision):
    import torch

    import paper_1904_11055_amd as ps
    N, width = 64, 0.25
    delta = fieldgen.gaussian_field(N, 5).astype(np.float32)
    half = torch.from_numpy(np.fft.rfftn(delta).astype(np.complex64))[None].to("cuda:0")
    plan = ps.Plan(N, order, nb, width, precision=precision, flags=ps.INPUT_HALF_SPECTRUM, device="cuda:0")
    at = np.flatnonzero((plan.tuples == np.array(tuple_)).all(axis=1))
    assert len(at) == 1
    g = np.random.default_rng(3).standard_normal(plan.n_closing)
    plan.shells(half)
    out = []
    for value in (0.0, np.nan):
        g[at[0]] = value
        out.append(plan.backward(torch.from_numpy(g)[None].to("cuda:0")).cpu().numpy()[0])
    plan.close()
    zero, nan = out
    assert np.all(np.isfinite(zero))
    shell = _shells(N, width)
    marred = set(tuple_) | {(s - 1 ^ 1) + 1 for s in tuple_}
    for s in range(1, nb + 1):
        modes = shell == s
        if s in tuple_:
            assert not np.any(np.isfinite(nan[modes].real))
        elif s not in marred:
            assert np.array_equal(nan[modes], zero[modes]), f"shell {s}"
