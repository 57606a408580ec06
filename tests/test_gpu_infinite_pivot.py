"""A matrix with an infinite diagonal element has no factor, wherever the element
stands: in the last row of a 64-wide block, or of the matrix, no later pivot shows it."""
import numpy as np
import pytest
import torch

from paper_2311_08050_amd import binding, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16"])
@pytest.mark.parametrize("n", [1, 16, 63, 64, 65, 128, 192, 200, 640])
def test_reported_in_range(n, prec):
    lib = binding.Library()
    spd = synth.random_spd(n, seed=n)
    rows = sorted({0, n // 2, max(0, n - 2), n - 1} | {i for i in (15, 16, 62, 63, 64, 127, 128, 191) if i < n})
    mats = []
    for i in rows:
        X = spd.copy()
        X[i, i] = np.inf
        mats.append(torch.as_tensor(X).cuda())
    mats.append(torch.as_tensor(spd).cuda())
    ld, info = lib.logdet(mats, prec=prec)
    for i, l, f in zip(rows, ld, info):
        assert f > 0 and i < f <= max(n, i + 2) and np.isnan(l), (i, l, f)
    assert info[-1] == 0 and np.isfinite(ld[-1])
