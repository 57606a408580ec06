"""The autotuner times the kernels that an evaluation runs: an FP32 batch with border
rows has its 128 x 128 updates on split BF16 operands, at 2.7 times the rate that the FP32
units bound the 64 x 64 ones to, and at order 6144 the updates are most of the time."""
import pytest

from paper_2311_08050_amd import binding

pytestmark = pytest.mark.gpu


def test_fp32_evaluations_keep_the_split_update():
    lib = binding.Library()
    cfg, times = lib.autotune([6144] * 4, [130] * 4, prec="fp32", reps=2)
    for nb in (256, 512, 1024):
        assert times[(nb, 128, 0)] < times[(nb, 64, 0)], times
    assert cfg[1] == 128
    assert lib.tune_get("fp32", 6144, 4) == cfg


@pytest.mark.parametrize("prec", ["fp32", "bf16"])
@pytest.mark.parametrize("ns,kbs", [([1, 700], [1, 130]), ([300, 1500], [0, 5]), ([900], [0])])
def test_shapes(ns, kbs, prec):
    """Orders below and above a panel, with and without border rows."""
    cfg, times = binding.Library().autotune(ns, kbs, prec=prec, reps=1)
    assert cfg in times and all(v > 0 for v in times.values())
