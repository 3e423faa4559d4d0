"""GPU: CAMPS factorisations under a caller's truncation threshold.

Circuits U, Pauli faults, U^dag with U a random Clifford+T network: a faulty
shot's P_acc is |<0|U^dag P U|0>|^2, often neither 0 nor 1.  Their residuals
have no Schmidt value below 0.03 of the largest, so a threshold up to there
drops nothing (the peak bonds stay those of the default threshold) and P_acc
must be the state vector's, as at the default: within 1e-10, the bound of the
other CAMPS tests.  A factorisation that leaves a small column unrotated loses
what it shares with a kept one, an error of first order in the threshold.
"""
import random

import numpy as np
import pytest

import paper_2609_19116_amd as msc
from paper_2609_19116_amd import results_numpy
from oracle import sampler as osamp
from oracle import statevector as sv
from oracle.ir import parse
from tests.helpers import say, to_dev

pytestmark = pytest.mark.gpu

INVERSE = {"H": "H", "S": "SDG", "T": "TDG", "CX": "CX", "CZ": "CZ"}


def _text(seed, n=8, layers=10):
    r = random.Random(seed)
    u = [("H", q) for q in range(1, n)]
    for _ in range(layers):
        for _ in range(6):
            g = r.choice(["H", "S", "CX", "CX", "CZ"])
            if g in ("CX", "CZ"):
                a = r.randrange(1, n - 1)
                u.append((g, a, a + 1) if r.random() >= 0.5 else (g, a + 1, a))
            else:
                u.append((g, r.randrange(1, n)))
        u.append(("T", r.randrange(1, n)))
    lines = [f"QUBITS {n}", "SEED 0", "TARGET T"] + [f"R {q}" for q in range(n)] + ["H 0", "T 0"]
    lines += [" ".join(map(str, g)) for g in u]
    lines += [f"DEP1 {q}" for q in range(1, n)]
    lines += [" ".join(map(str, (INVERSE[g[0]],) + g[1:])) for g in reversed(u)]
    return "\n".join(lines + [f"M {q}" for q in range(1, n)]) + "\n"


def test_camps_threshold_below_the_spectrum_changes_nothing():
    import torch
    assert torch.cuda.is_available()
    ctx = msc.Ctx(0)
    n = 24
    w = (1 + np.arange(n) % 3).astype(np.int32)
    between = 0
    for seed in range(8):
        text = _text(seed)
        circ = msc.Circuit(text)
        say(f"camps truncation circuit {seed}")
        circ.calibrate(ctx)
        csr = msc.sample_faults(circ, 11 + seed, 0, n, weights=w)
        dev = to_dev(*csr)
        oc = parse(text)
        ref = np.array([sv.run_shot(oc, f).p_acc for f in osamp.csr_to_dicts(*csr)])
        base = results_numpy(msc.simulate_camps(ctx, circ, *dev))
        between += int(((ref > 1e-3) & (ref < 0.999)).sum())
        for tau in (0.0, 1e-3, 1e-2, 3e-2):
            res = results_numpy(msc.simulate_camps(ctx, circ, *dev, tau_trunc=tau))
            assert not (res["status"] & msc.SHOT_NOCONV).any(), (seed, tau)
            assert np.array_equal(res["chi_peak"], base["chi_peak"]), (seed, tau)
            assert np.abs(res["p_acc"] - ref).max() < 1e-10, (seed, tau)
    assert between > 20
    ctx.close()
