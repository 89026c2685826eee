"""The shell fields of the narrow inverse column blocks are those of the wide ones bit for bit.

The digests were taken with column blocks of elems / N pencils, which the passes used before
they were narrowed.  They belong to the code that hipcc of ROCm 7.2 makes; under a compiler that
contracts other multiply-adds the fields may differ from them by 1 ulp, which is no error.
"""
import hashlib

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.timeout(120)
@pytest.mark.parametrize("N,order,nb,width,digest", [
    (32, 2, 3, 4.0, "660ca61e30997879"),
    (64, 2, 3, 8.0, "92a5045f10dd51b5"),
    (64, 3, 16, 1.0, "9dc6a6cd2e82af93"),
    (128, 2, 3, 16.0, "7812404518ac747e"),
    (128, 3, 24, 1.0, "84b8650c62ccd924"),
    (256, 2, 3, 32.0, "6e38970522c1feb4"),
    (256, 3, 20, 2.0, "b2c5550922ea4e3e"),
])
def test_fields_of_the_wide_blocks(gpu, N, order, nb, width, digest):
    """Whole numbers as the half spectrum, so that no input transform takes part."""
    import torch

    import paper_1904_11055_amd as ps
    rng = np.random.default_rng(N)
    half = rng.integers(-1024, 1025, (N, N, N // 2 + 1, 2)).astype(np.float32).view(np.complex64)[..., 0]
    plan = ps.Plan(N, order, nb, width, precision=ps.FP32, flags=ps.INPUT_HALF_SPECTRUM, device="cuda:0")
    plan.shells(torch.from_numpy(half)[None].to("cuda:0"))
    fields = plan.fields().cpu().numpy()
    plan.close()
    assert hashlib.sha256(fields.tobytes()).hexdigest()[:16] == digest
