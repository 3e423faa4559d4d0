"""GPU: which kernel takes a run's shots, over the bond caps a caller may set.

Noiseless bonds: 16 (17 qubits), 32 (49 qubits, snake layout), 64 (81 qubits)
and 128 (49 qubits, rainbow layout).
"""
import numpy as np
import pytest

import paper_2609_19116_amd as msc
from paper_2609_19116_amd import MSC_FP32, MSC_FP64, results_numpy
from tests.helpers import say, to_dev
from workloads.circuits import config_circuit

pytestmark = pytest.mark.gpu

FIELDS = ["p_acc", "infid", "disc_weight", "chi_peak", "status", "rejected_at", "fail", "n2q",
          "flops", "sweeps"]
_CIRC = {}


@pytest.fixture(scope="module")
def ctx():
    import torch
    assert torch.cuda.is_available()
    c = msc.Ctx(0)
    yield c
    c.close()


def _circuit(ctx, name):
    if name not in _CIRC:
        c = msc.Circuit(config_circuit(name).text)
        say(f"calibrate {name}")
        c.calibrate(ctx)
        _CIRC[name] = c
    return _CIRC[name]


@pytest.mark.parametrize("precision", [MSC_FP64, MSC_FP32])
@pytest.mark.parametrize("prefix", [False, True])
@pytest.mark.parametrize("chi_max", [8, 16, 24, 31])
def test_cap_below_the_noiseless_bond_keeps_the_workgroup_kernel(ctx, chi_max, prefix, precision):
    # what a binding cap drops among equal singular values follows the
    # factorisation's basis, so every bit of these records belongs to one kernel
    c = _circuit(ctx, "c3")
    assert c.noiseless()["chi_peak"] == 32
    n = 12
    off, ch, pa = to_dev(*msc.sample_faults(c, 0x5EED0211, 0, n,
                                            weights=(np.arange(n) % 4).astype(np.int32)))
    say(f"c3 chi_max={chi_max} prefix={prefix} precision={precision}")
    kw = dict(precision=precision, chi_max=chi_max, prefix=prefix)
    a = results_numpy(msc.simulate(ctx, c, off, ch, pa, **kw))
    b = results_numpy(msc.simulate(ctx, c, off, ch, pa, wave_chi=-1, **kw))
    assert np.any(a["status"] & msc.SHOT_CHI_CAP)
    for f in FIELDS:
        assert np.array_equal(a[f], b[f]), f
