"""GPU: which kernel takes a run's shots, over the bond caps a caller may set.

Noiseless bonds: 16 (17 qubits), 32 (49 qubits, snake layout), 64 (81 qubits)
and 128 (49 qubits, rainbow layout).
"""
import json
import os

import numpy as np
import pytest

import paper_2609_19116_amd as msc
from paper_2609_19116_amd import MSC_FP32, MSC_FP64, results_numpy
from oracle import statevector as sv
from oracle.ir import parse
from tests.helpers import say, to_dev
from tests.test_gpu_parity import TOL, _compare
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


@pytest.mark.parametrize("name,kernel,slot", [
    ("c1", "mps_fast_wave_kernel", 16), ("c1_ghz", "mps_wave_kernel", 16),
    ("c3", "mps_fast_mid_kernel", 32), ("c4", "mps_fast_group_kernel", 128),
    ("c3_rainbow", "mps_fast_group_kernel", 128)])
def test_stats_name_the_kernel(ctx, name, kernel, slot):
    c = _circuit(ctx, name)
    off, ch, pa = to_dev(*msc.sample_faults(c, 0x5EED0213, 0, 3,
                                            weights=np.array([0, 1, 1], dtype=np.int32)))
    say(f"{name} shot kernel")
    res = results_numpy(msc.simulate(ctx, c, off, ch, pa, precision=MSC_FP32))
    st = ctx.engine_stats()
    assert (st["shot_kernel"], st["slot_chi"]) == (kernel, slot)
    assert st["slots"] >= 3 and st["slot_retries"] == 0
    alone = results_numpy(msc.simulate(ctx, c, off, ch, pa, precision=MSC_FP32, wave_chi=-1))
    st = ctx.engine_stats()
    assert (st["shot_kernel"], st["slot_chi"], st["slot_retries"]) == ("mps_kernel", 256, 0)
    # a kernel that ran nothing would still have left its name
    for r in (res, alone):
        assert np.all(r["status"] & (msc.SHOT_DONE | msc.SHOT_REJECTED))
    # gauge-independent counts (controlled-S circuits: their updates follow the
    # basis of equal singular values, here that of one and the same sweep)
    for f in ("chi_peak", "n2q", "flops", "status", "rejected_at", "fail"):
        assert np.array_equal(res[f], alone[f]), f


@pytest.mark.parametrize("precision", [MSC_FP64, MSC_FP32])
@pytest.mark.parametrize("name,chi", [("c4", 64), ("c3_rainbow", 128)])
def test_group_kernel_matches_stored_oracle_values(ctx, name, chi, precision):
    # bonds 64 and 128 at the default options: theta in LDS and in scratch,
    # Gram matrices of up to sixteen tiles a side
    import torch
    with open(os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden",
                           f"large_chi_{name}.json")) as f:
        g = json.load(f)
    c = _circuit(ctx, name)
    w = np.full(g["candidates"], g["weight_of_every_shot"], dtype=np.int32)
    csr = msc.sample_faults(c, int(g["seed"], 16), 0, len(w), weights=w)
    ref = np.array([(s["p_acc"], s["infid"], s["rejected_at"]) for s in g["shots"]])
    idx = torch.tensor([s["shot"] for s in g["shots"]], dtype=torch.int64, device="cuda")
    say(f"{name} stored shots precision={precision}")
    res = results_numpy(msc.simulate(ctx, c, *to_dev(*csr), shot_idx=idx, precision=precision))
    assert ctx.engine_stats()["shot_kernel"] == "mps_fast_group_kernel"
    _compare(res, ref, TOL[precision])
    assert np.all(res["chi_peak"][ref[:, 0] > 0] >= chi)
    assert not np.any(res["status"] & (msc.SHOT_CHI_CAP | msc.SHOT_NOCONV))


def _nested_pairs(m, depth=1):
    """m nested Bell pairs (bond 2^m between their halves) around two qubits
    that CX entangles only in shots where a fault between (T H)^depth and its
    inverse leaves the first one off |0>: those double the bond."""
    n = 2 * m + 3
    a, b = m, m + 1
    pairs = [(i, n - 2 - i) for i in range(m)]
    ops = [f"H {n - 1}", f"T {n - 1}"] + [f"H {a}", f"T {a}"] * depth
    ops += [f"DEP1 {a}"] + [f"TDG {a}", f"H {a}"] * depth
    for i, j in pairs:
        ops += [f"H {i}", f"CX {i} {j}"]
    ops += ["DEP1 0", f"CX {a} {b}", f"CX {a} {b}"]
    for i, j in reversed(pairs):
        ops += [f"CX {i} {j}", f"H {i}"]
    return "\n".join([f"QUBITS {n}", f"SEED {n - 1}", "TARGET T"] + [f"R {q}" for q in range(n)]
                     + ops + [f"M {q}" for q in range(n - 1)]) + "\n"


def _fault_list(faults):
    off = np.concatenate([[0], np.cumsum([len(f) for f in faults])]).astype(np.int64)
    return (off, np.array([k for f in faults for k in f], dtype=np.int32),
            np.array([v for f in faults for v in f.values()], dtype=np.uint8))


@pytest.mark.parametrize("precision", [MSC_FP64, MSC_FP32])
@pytest.mark.parametrize("m,kernel", [(4, "mps_fast_wave_kernel"), (5, "mps_fast_mid_kernel"),
                                      (7, "mps_fast_group_kernel")])
def test_shots_that_outgrow_their_slot(ctx, m, kernel, precision):
    # the noiseless bond is the slots' cap: faulty shots of twice the bond are
    # run again by the workgroup kernel, once each, and counted
    text = _nested_pairs(m)
    c = msc.Circuit(text)
    say(f"nested pairs m={m} precision={precision}")
    c.calibrate(ctx)
    assert c.noiseless()["chi_peak"] == 2 ** m
    faults = [{}, {0: 1}, {0: 2}, {0: 3}, {1: 1}, {0: 1, 1: 3}, {0: 1}, {}]
    off, ch, pa = _fault_list(faults)
    oc = parse(text)
    ref = np.array([(r.p_acc, r.infid, r.rejected_at) for r in (sv.run_shot(oc, f) for f in faults)])
    res = results_numpy(msc.simulate(ctx, c, *to_dev(off, ch, pa), precision=precision))
    st = ctx.engine_stats()
    assert (st["shot_kernel"], st["slot_chi"]) == (kernel, 2 ** m)
    wide = res["chi_peak"] > 2 ** m
    assert list(wide) == [f.get(0, 2) != 2 for f in faults]
    assert st["slot_retries"] == wide.sum()
    assert st["wave_retries"] == (wide.sum() if m == 4 else 0)
    _compare(res, ref, TOL[precision])
    # the same from checkpoints of the noiseless run
    pf = results_numpy(msc.simulate(ctx, c, *to_dev(off, ch, pa), precision=precision, prefix=True))
    assert ctx.engine_stats()["slot_retries"] == wide.sum()
    for f in FIELDS[:7]:
        assert np.array_equal(res[f], pf[f]), f


@pytest.mark.parametrize("precision", [MSC_FP64, MSC_FP32])
@pytest.mark.parametrize("m,kernel", [(5, "mps_fast_mid_kernel"), (7, "mps_fast_group_kernel")])
def test_a_full_slot_is_no_bond_cap(ctx, m, kernel, precision):
    # an X fault at depth 3 leaves amplitudes 0.146 and 0.989, Schmidt values in
    # the ratio 0.148 on top of the pairs' equal ones: a threshold of 0.6 drops
    # the smaller half, so the bond stays at the slots' cap, which cut nothing,
    # and chi_max (256) is far away
    c = msc.Circuit(_nested_pairs(m, depth=3))
    say(f"full slot m={m} precision={precision}")
    c.calibrate(ctx)
    assert c.noiseless()["chi_peak"] == 2 ** m
    dev = to_dev(*_fault_list([{}, {0: 1}, {0: 1, 1: 1}, {0: 1}]))
    kw = dict(precision=precision, tau_trunc=0.6)
    res = results_numpy(msc.simulate(ctx, c, *dev, **kw))
    st = ctx.engine_stats()
    assert (st["shot_kernel"], st["slot_chi"], st["slot_retries"]) == (kernel, 2 ** m, 0)
    assert np.all(res["disc_weight"][1:] > 0.01) and np.all(res["chi_peak"] == 2 ** m)
    assert not np.any(res["status"] & msc.SHOT_CHI_CAP)
    ref = results_numpy(msc.simulate(ctx, c, *dev, wave_chi=-1, **kw))
    for f in ("status", "chi_peak", "rejected_at", "fail", "n2q", "flops"):
        assert np.array_equal(res[f], ref[f]), f
    np.testing.assert_allclose(res["p_acc"], ref["p_acc"], rtol=2 * TOL[precision], atol=0)
