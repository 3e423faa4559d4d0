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


@pytest.mark.parametrize("precision", [MSC_FP64, MSC_FP32])
@pytest.mark.parametrize("prefix", [False, True])
def test_every_cap_that_holds_the_bond_gives_the_same_records(ctx, prefix, precision):
    # slots of any cap from the noiseless bond (64) on: the cap is where a slot
    # ends, not part of a result (66 to 124: theta sides that are no multiple
    # of 16)
    c = _circuit(ctx, "c4")
    assert c.noiseless()["chi_peak"] == 64
    off, ch, pa = to_dev(*msc.sample_faults(c, 0x5EED0212, 0, 3,
                                            weights=np.array([0, 1, 2], dtype=np.int32)))
    kw = dict(precision=precision, prefix=prefix)
    ref = results_numpy(msc.simulate(ctx, c, off, ch, pa, **kw))
    assert not np.any(ref["status"] & msc.SHOT_CHI_CAP)
    for chi_max in (64, 65, 66, 74, 82, 91, 100, 108, 116, 124, 127, 128, 129):
        say(f"c4 chi_max={chi_max} prefix={prefix} precision={precision}")
        a = results_numpy(msc.simulate(ctx, c, off, ch, pa, chi_max=chi_max, **kw))
        for f in FIELDS:
            assert np.array_equal(a[f], ref[f]), (f, chi_max)
