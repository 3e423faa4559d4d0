"""Edges of the matrix-core shot kernels, the screen and the FP32 contraction.

Shot counts around the number of shots of a workgroup (four of bond 16, seven
of bond 32, one of bond 128), screens whose blocks take each of their routes
(several runs of faults, more faults of survivors than the list holds, no hash
table, odd sizes), and contractions whose tile counts
are not multiples of the XCD count.

Tolerances: a shot result is within TOL[precision] of the oracle in either
shot kernel, so two kernels are within twice that of each other; the screen is
exact; a contraction of K = chi complex FP32 products is off by at most
about 2 sqrt(K) roundings of 2^-24, below 1e-5 for every K here.
"""
import numpy as np
import pytest

import paper_2609_19116_amd as msc
from paper_2609_19116_amd import MSC_FP32, MSC_FP64, results_numpy
from tests.helpers import oracle_discards, say, to_dev
from tests.test_gpu_parity import TOL
from workloads.circuits import config_circuit

pytestmark = pytest.mark.gpu

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
@pytest.mark.parametrize("name,sizes", [("tiny", (1, 3, 4, 5)), ("c1", (1, 4, 9)),
                                        ("c3", (1, 6, 7, 8, 15)), ("c4", (1, 2))])
def test_matrix_core_shots_match_workgroup_kernel(ctx, name, sizes, precision):
    c = _circuit(ctx, name)
    n = max(sizes)
    w = np.arange(n) % 4
    off, ch, pa = to_dev(*msc.sample_faults(c, 0x5EED0201, 0, n, weights=w.astype(np.int32)))
    say(f"workgroup kernel {name} precision={precision} n={n}")
    ref = results_numpy(msc.simulate(ctx, c, off, ch, pa, precision=precision, wave_chi=-1))
    for k in sizes:
        say(f"matrix cores {name} precision={precision} n={k}")
        got = results_numpy(msc.simulate(ctx, c, off[:k + 1], ch, pa, precision=precision))
        r = ref[:k]
        for f in ("rejected_at", "fail", "status"):
            assert np.array_equal(got[f], r[f]), (f, k)
        acc = r["p_acc"] > 0
        assert np.all(got["p_acc"][~acc] == 0)
        scale = np.maximum(r["infid"], 1 - r["infid"])[acc]
        assert np.all(np.abs(got["p_acc"] - r["p_acc"])[acc] <= 2 * TOL[precision] * r["p_acc"][acc])
        assert np.all(np.abs(got["infid"] - r["infid"])[acc] <= 2 * TOL[precision] * scale)


def test_checkpoints_belong_to_the_kernel_that_recorded_them(ctx):
    # bond 32: an explicit wave_chi 32 runs the general wavefront kernel, the
    # automatic choice the matrix-core kernel of the same cap; a forked run
    # repeats its own kernel's bits whichever recorded checkpoints before
    c = msc.Circuit(config_circuit("c3").text)
    say("calibrate c3")
    c.calibrate(ctx)
    n = 24
    off, ch, pa = to_dev(*msc.sample_faults(c, 0x5EED0207, 0, n,
                                            weights=(np.arange(n) % 3).astype(np.int32)))
    kw = dict(precision=MSC_FP32)
    for chi in (0, 32, 0):
        say(f"forked and plain wave_chi={chi}")
        a = results_numpy(msc.simulate(ctx, c, off, ch, pa, wave_chi=chi, **kw))
        b = results_numpy(msc.simulate(ctx, c, off, ch, pa, wave_chi=chi, prefix=True, **kw))
        for f in ("p_acc", "infid", "chi_peak", "status", "rejected_at", "fail"):
            assert np.array_equal(a[f], b[f]), (chi, f)


def _check_screen(ctx, c, text, csr):
    from oracle.ir import parse
    n = len(csr[0]) - 1
    keep = ~oracle_discards(parse(text), csr)
    say(f"screen n={n} faults={csr[0][-1]} survivors={keep.sum()}")
    bits, idx, cnt = msc.prescreen(ctx, c, *to_dev(*csr))
    b = np.unpackbits(bits.cpu().numpy().view(np.uint8), bitorder="little")
    assert np.array_equal(b[:n].astype(bool), keep)
    assert not b[n:].any()
    assert cnt == keep.sum()
    assert np.array_equal(idx.cpu().numpy(), np.nonzero(keep)[0])


def _tile(csr, picks):
    off, ch, pa = csr
    rows = [np.arange(off[i], off[i + 1]) for i in picks]
    at = np.concatenate(rows).astype(np.int64)
    new = np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(off.dtype)
    return new, ch[at], pa[at]


@pytest.mark.parametrize("name,n,weight", [
    ("c1", 1, 2), ("c1", 63, 1), ("c1", 257, 3), ("c1", 1023, 2), ("c1", 1025, 2),
    ("c1", 1030, 4),            # blocks of exactly one run of 1024 faults
    ("c1", 1100, 5),            # two runs: survivors walked
    ("c1_ghz", 1024, 13),       # four runs, three-qubit codes
    ("tiny", 2049, 0),          # no faults at all
])
def test_screen_block_edges(ctx, name, n, weight):
    text = config_circuit(name).text
    c = msc.Circuit(text)
    w = np.full(n, weight, dtype=np.int32)
    _check_screen(ctx, c, text, msc.sample_faults(c, 0x5EED0202, 0, n, weights=w))


@pytest.mark.parametrize("kind", ["every", "list", "mixed"])
def test_screen_many_survivors_with_faults(ctx, kind):
    text = config_circuit("c1").text
    c = msc.Circuit(text)
    n = 4000
    csr = msc.sample_faults(c, 0x5EED0203, 0, n, weights=(1 + np.arange(n) % 4).astype(np.int32))
    from oracle.ir import parse
    dead = oracle_discards(parse(text), csr)
    wt = np.diff(csr[0])
    alive, heavy = np.nonzero(~dead)[0], np.nonzero(~dead & (wt >= 3))[0]
    gone = np.nonzero(dead & (wt == 1))[0]
    assert len(alive) > 20 and len(heavy) > 3
    m = 1500
    if kind == "every":          # every shot survives with faults
        picks = np.resize(alive, m)
    elif kind == "list":         # the same, above 512 faults of survivors in a block
        picks = np.resize(heavy, m)
    else:                        # a few survivors among the others
        picks = np.where(np.arange(m) % 20 == 0, np.resize(alive, m), np.resize(gone, m))
    _check_screen(ctx, c, text, _tile(csr, picks))


def test_screen_without_hash_table(ctx):
    # three-qubit channels take 64 entries each: 131073 channels pass the
    # table's limit of 2^23 entries, and every shot is walked
    lines = config_circuit("tiny_ghz").text.splitlines()
    at = next(i for i, x in enumerate(lines) if x.startswith("M "))
    lines[at:at] = ["DEP1 " + lines[at].split()[1]] * 131100
    text = "\n".join(lines) + "\n"
    c = msc.Circuit(text)
    n = 700
    _check_screen(ctx, c, text, msc.sample_faults(c, 0x5EED0204, 0, n,
                                                  weights=(np.arange(n) % 3).astype(np.int32)))


@pytest.mark.parametrize("chi,batch", [(64, 1), (128, 5), (192, 3), (320, 1)])
def test_contract_fp32_tile_counts(ctx, chi, batch):
    import torch
    from workloads.tensors import random_twosite
    A, B, G, Ac, Bc, _ = random_twosite(chi, batch, 0x5EED0205, "haar")
    Gc = G.reshape(4, 4, 2).astype(np.float64)
    Gc = (Gc[..., 0] + 1j * Gc[..., 1]).reshape(2, 2, 2, 2)
    th = torch.zeros(batch * 2 * (2 * chi) ** 2, dtype=torch.float32).cuda()
    dA, dB, dG = to_dev(A, B, G)
    say(f"contract fp32 chi={chi} batch={batch}")
    msc.twosite_contract(ctx, chi, batch, dA, dB, dG, th, precision=MSC_FP32)
    got = th.cpu().numpy().reshape(batch, 2, 2 * chi, 2 * chi).astype(np.float64)
    for b in range(batch):
        T = (Ac[b] @ Bc[b]).reshape(chi, 2, 2, chi)
        ref = np.einsum("ijkl,aklb->aijb", Gc, T).reshape(2 * chi, 2 * chi)
        err = np.linalg.norm(got[b, 0] + 1j * got[b, 1] - ref) / np.linalg.norm(ref)
        assert err < 1e-5, (b, err)


@pytest.mark.parametrize("name,n", [("tiny", 5), ("c3", 9), ("c4", 2)])
def test_camps_bond_routes_match_mps(ctx, name, n):
    # from trivial moves of product bonds to factorisations in LDS
    c = _circuit(ctx, name)
    w = (np.arange(n) % 3).astype(np.int32)
    off, ch, pa = to_dev(*msc.sample_faults(c, 0x5EED0206, 0, n, weights=w))
    say(f"camps {name} n={n}")
    a = results_numpy(msc.simulate_camps(ctx, c, off, ch, pa))
    b = results_numpy(msc.simulate(ctx, c, off, ch, pa, precision=MSC_FP64, wave_chi=-1))
    assert np.array_equal(a["rejected_at"], b["rejected_at"])
    assert np.array_equal(a["fail"], b["fail"])
    assert np.allclose(a["p_acc"], b["p_acc"], atol=1e-9, rtol=0)
    acc = b["p_acc"] > 0
    assert np.allclose(a["infid"][acc], b["infid"][acc], atol=1e-9, rtol=0)
