"""Performance cases of the shot simulator: what a study of cultivation
circuits runs on one GPU, through the package's public entry points.

A case is one of five kinds of call:

- ``batch``: ``run_batch``, the whole path of one batch (fault sampling,
  offline screen, shots, sums per weight), as a sweep over error rates
  calls it again and again;
- ``shots``: ``simulate`` on a caller's own fault list (subset sampling,
  replayed shots, a few patterns under study);
- ``camps``: ``simulate_camps`` on the survivors of a fault list;
- ``screen``: ``sample_faults_device`` and ``prescreen``, the part of a
  large study that runs over every shot drawn;
- ``contract``: ``twosite_contract`` on the caller's tensors.

Per-shot records are returned field by field.  Two fields are left out:
``disc_weight`` and ``sweeps`` say how the factorisations went (the summed
squares of numerical zeros, the number of sweeps), not what they computed.
The infidelity is returned as the fidelity 1 - infid, the quantity its
accuracy refers to.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2609_19116_amd as msc
from workloads.circuits import config_circuit, make_circuit

# The 49-qubit circuit's order from the qubit-order search (three starts of
# 128 evaluations from the snake order, then four rounds that continue from
# the best): the layout its batches run on.
SEARCHED_49Q = [9, 0, 8, 1, 6, 5, 3, 4, 2, 7, 12, 11, 13, 17, 18, 14, 10, 15, 20, 16, 19, 21, 26,
                25, 24, 23, 22, 27, 29, 28, 32, 31, 33, 34, 30, 35, 38, 37, 39, 36, 41, 46, 40,
                45, 44, 43, 42, 47, 48]

# circuit -> (workload name, order, noise channels M, flops of the two-site
# updates of one fault-free shot from its start to its end), the latter as
# the records count them (contraction, Gram matrix, projection and
# eigen-decomposition at the realised shapes)
CIRCUITS = {
    "7q": ("tiny", None, 55, 2.1e5),
    "17q": ("c1", None, 292, 1.04e7),
    "17q_ghz": ("c1_ghz", None, 388, 7.4e7),
    "49q": ("c3", SEARCHED_49Q, 1249, 1.98e8),
    "49q_snake": ("c3", None, 1249, 6.4e8),
    "81q": ("81q_short", None, 1180, 3.8e10),
    "81q_full": ("c4", None, 2869, 7.0e10),
}
WMAX = 64          # bins of a batch: weights 0 .. 64
PRECISION = {"fp64": msc.MSC_FP64, "fp32": msc.MSC_FP32, "bf16x3": msc.MSC_BF16X3}


def listed():
    return [
        # one step of a large study: the 49-qubit circuit at the error rate
        # the method is quoted at, enough shots to fill the GPU
        dict(name="batch_49q", kind="batch", circuit="49q", precision="fp32", shots=1 << 19,
             p=1e-3, space_time=False, prefix=True),
        # the same circuit in a short call: a first look at an error rate
        dict(name="batch_49q_small", kind="batch", circuit="49q", precision="fp32", shots=1000,
             p=1e-3, space_time=False, prefix=True),
        # no layout search: the snake order, whose bond is twice as large
        dict(name="batch_49q_snake", kind="batch", circuit="49q_snake", precision="fp32",
             shots=20000, p=5e-4, space_time=False, prefix=True),
        # the space-time accounting (no screen: every shot is simulated), in
        # double precision
        dict(name="batch_17q_space_time", kind="batch", circuit="17q", precision="fp64",
             shots=10007, p=2e-3, space_time=True, prefix=True),
        # subset sampling with a fixed number of faults per shot, every shot
        # simulated from the start
        dict(name="shots_17q_subset", kind="shots", circuit="17q", precision="fp64", shots=65536,
             w_max=4, p=0.0, survivors=0, prefix=False),
        # a list of ordinary shots, in single precision
        dict(name="shots_17q", kind="shots", circuit="17q", precision="fp32", shots=1000, w_max=-1,
             p=2e-3, survivors=0, prefix=False),
        # a handful of fault patterns under study
        dict(name="shots_17q_few", kind="shots", circuit="17q", precision="fp64", shots=4,
             w_max=4, p=0.0, survivors=0, prefix=False),
        # the 81-qubit patch with one T layer, at bond dimension 64
        dict(name="shots_81q", kind="shots", circuit="81q", precision="fp32", shots=2500, w_max=-1,
             p=5e-4, survivors=256, prefix=True),
        # the Clifford-augmented engine on the survivors of a batch
        dict(name="camps_49q", kind="camps", circuit="49q_snake", precision="fp64", shots=1024,
             w_max=-1, p=1e-3, survivors=256, prefix=True),
        # drawing and screening the shots of the largest circuit
        dict(name="screen_81q", kind="screen", circuit="81q_full", shots=(1 << 24) - 5, p=1e-3),
        # fixed-shape two-site contractions at the largest bond of a run
        dict(name="contract_fp32", kind="contract", precision="fp32", chi=256, batch=192),
        dict(name="contract_bf16x3", kind="contract", precision="bf16x3", chi=256, batch=384),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["batch", "batch", "batch", "shots", "shots", "camps", "screen", "contract"])
    if kind == "batch":
        circuit = rng.choice(["17q", "17q_ghz", "49q", "49q", "49q_snake"])
        # shots that are simulated rather than screened cost most
        top = {"17q": 30000, "17q_ghz": 3000, "49q": 200000, "49q_snake": 15000}[circuit]
        space_time = rng.random() < 0.25
        prefix = rng.random() < 0.8
        precision = rng.choice(["fp32", "fp32", "fp64"])
        if space_time or not prefix:
            top //= 8
        if precision == "fp64":
            top //= 2
        return dict(kind="batch", circuit=circuit, precision=precision,
                    shots=_log_int(rng, 100, top), p=round(10 ** rng.uniform(-3.5, -2.6), 7),
                    space_time=space_time, prefix=prefix)
    if kind == "shots":
        circuit = rng.choice(["7q", "17q", "17q_ghz", "49q", "81q"])
        top = {"7q": 30000, "17q": 20000, "17q_ghz": 1000, "49q": 2000, "81q": 100}[circuit]
        screened = circuit in ("49q", "81q")
        n = _log_int(rng, 24 if screened else 4, top)
        subset = rng.random() < 0.5 or n < 300      # few shots: of a fixed number of faults
        return dict(kind="shots", circuit=circuit, precision=rng.choice(["fp32", "fp64"]),
                    shots=24 * n + 64 if screened else n,
                    w_max=rng.randint(2, 4) if subset and not screened else -1,
                    p=round(10 ** rng.uniform(-3.5, -2.8), 7),
                    survivors=n if screened else 0, prefix=rng.random() < 0.5)
    if kind == "camps":
        n = _log_int(rng, 24, 200)
        return dict(kind="camps", circuit=rng.choice(["17q", "49q_snake"]), precision="fp64",
                    shots=24 * n + 64, w_max=-1, p=round(10 ** rng.uniform(-3.5, -2.8), 7),
                    survivors=n, prefix=rng.random() < 0.8)
    if kind == "screen":
        return dict(kind="screen", circuit=rng.choice(["17q", "49q", "81q_full"]),
                    shots=_log_int(rng, 1000, 1 << 24), p=round(10 ** rng.uniform(-3.5, -2.6), 7))
    chi = rng.choice([64, 128, 192, 256, 320, 448, 512])
    precision = rng.choice(["fp32", "bf16x3"])
    top = (150 if precision == "fp32" else 300) * (256 / chi) ** 3
    return dict(kind="contract", precision=precision, chi=chi,
                batch=_log_int(rng, 1, max(2, min(2000, top))))


# ---------------------------------------------------------------------------
# what a user's program holds before the call

_CTX = []


def _ctx():
    """The program's one context (stream and scratch)."""
    if not _CTX:
        _CTX.append(msc.Ctx(0))
    return _CTX[0]


def _text(name):
    workload = CIRCUITS[name][0]
    if workload == "81q_short":
        return make_circuit("unrot", 5, plain_rounds=1, t_layers=1, framed_rounds=2,
                            final_rounds=0).text
    return config_circuit(workload).text


def _circuit(name, calibrate=True):
    c = msc.Circuit(_text(name), order=CIRCUITS[name][1])
    if calibrate:
        c.calibrate(_ctx())
    return c


def _channels(text):
    """Number of Pauli codes of each noise channel, in text order."""
    codes = {"XERR": 2, "DEP1": 4, "DEP2": 16, "DEP3": 64}
    return np.array([codes[ln.split()[0]] for ln in text.splitlines()
                     if ln and ln.split()[0] in codes], dtype=np.int64)


def _faults(case, seed):
    """Fault list (CSR) of the case: per shot w distinct channels in
    ascending order with a uniform non-identity Pauli each; w uniform in
    0 .. w_max, or w ~ Bin(M, p)."""
    codes = _channels(_text(case["circuit"]))
    M, n = len(codes), case["shots"]
    rng = np.random.default_rng(seed)
    w = rng.integers(0, case["w_max"] + 1, n) if case["w_max"] >= 0 else rng.binomial(M, case["p"], n)
    off = np.zeros(n + 1, dtype=np.int64)
    np.cumsum(w, out=off[1:])
    chan = np.zeros(off[-1], dtype=np.int32)
    for k in np.unique(w):
        rows = np.nonzero(w == k)[0]
        if k == 0:
            continue
        pick = np.sort(rng.integers(0, M, (len(rows), k)), axis=1)
        while True:
            again = (pick[:, 1:] == pick[:, :-1]).any(axis=1)
            if not again.any():
                break
            pick[again] = np.sort(rng.integers(0, M, (int(again.sum()), k)), axis=1)
        chan[off[rows][:, None] + np.arange(k)[None, :]] = pick
    pauli = (1 + rng.integers(0, codes[chan] - 1)).astype(np.uint8)
    return off, chan, pauli


def prepare(case, seed):
    kind = case["kind"]
    if kind == "contract":
        chi, batch = case["chi"], case["batch"]
        A, B, G = _tensors(case, seed)
        theta = torch.empty(batch, 2, 2 * chi, 2 * chi, dtype=torch.float32, device="cuda")
        return dict(case=case, A=A, B=B, G=G, theta=theta)
    st = dict(case=case, circ=_circuit(case["circuit"], kind != "screen"), seed=seed)
    if kind == "screen":
        # the study's own lists, which every chunk of shots is collected in
        n = case["shots"]
        mean = n * CIRCUITS[case["circuit"]][2] * case["p"]
        cap = int(mean + 10 * math.sqrt(mean) + 64)
        st["chan"] = torch.full((cap,), -1, dtype=torch.int32, device="cuda")
        st["pauli"] = torch.zeros(cap, dtype=torch.uint8, device="cuda")
        st["idx"] = torch.full((n,), -1, dtype=torch.int64, device="cuda")
    if kind in ("shots", "camps"):
        off, chan, pauli = (torch.from_numpy(a).cuda() for a in _faults(case, seed))
        idx = None
        if case["survivors"]:
            _, idx, _ = msc.prescreen(_ctx(), st["circ"], off, chan, pauli)
            idx = idx[: case["survivors"]].contiguous()
        st.update(off=off, chan=chan, pauli=pauli, idx=idx)
    return st


def _tensors(case, seed):
    """Normalised complex Gaussian site tensors and a random unitary gate."""
    chi, batch = case["chi"], case["batch"]
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    A = torch.randn(batch, 2, 2 * chi, chi, generator=g, device="cuda", dtype=torch.float32)
    B = torch.randn(batch, 2, chi, 2 * chi, generator=g, device="cuda", dtype=torch.float32)
    A /= A.flatten(1).norm(dim=1).view(-1, 1, 1, 1)
    B /= B.flatten(1).norm(dim=1).view(-1, 1, 1, 1)
    rng = np.random.default_rng(seed)
    q, r = np.linalg.qr(rng.standard_normal((4, 4)) + 1j * rng.standard_normal((4, 4)))
    q = q * (np.diag(r) / np.abs(np.diag(r)))
    G = torch.from_numpy(np.stack([q.real, q.imag], axis=-1).astype(np.float32).reshape(-1)).cuda()
    return A, B, G


def _records(out):
    """The records' fields, as views of the device buffer."""
    f8, i8 = out.view(torch.float64).view(-1, 8), out.view(torch.int64).view(-1, 8)
    i4 = out.view(torch.int32).view(-1, 16)
    return dict(p_acc=f8[:, 0], fidelity=1.0 - f8[:, 1], chi_peak=i4[:, 6], status=i4[:, 7],
                rejected_at=i4[:, 8], fail=i4[:, 9], n2q=i8[:, 5], flops=f8[:, 6])


def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "batch":
        bins, stats = msc.run_batch(_ctx(), st["circ"], st["seed"], 0, case["shots"], case["p"],
                                    n_bins=WMAX + 1, precision=PRECISION[case["precision"]],
                                    prefix=case["prefix"], space_time=case["space_time"])
        out = {k: stats[k] for k in ("nnz", "n_survivors", "n_accepted", "n2q", "flops",
                                     "chi_peak", "status_or")}
        out["bins"] = bins
        if case["space_time"]:
            out["reach"] = stats["surv_bins"]
        return out
    if kind == "shots":
        return _records(msc.simulate(_ctx(), st["circ"], st["off"], st["chan"], st["pauli"],
                                     shot_idx=st["idx"], precision=PRECISION[case["precision"]],
                                     prefix=case["prefix"]))
    if kind == "camps":
        return _records(msc.simulate_camps(_ctx(), st["circ"], st["off"], st["chan"], st["pauli"],
                                           shot_idx=st["idx"], prefix=case["prefix"]))
    if kind == "screen":
        off, chan, pauli = msc.sample_faults_device(_ctx(), st["circ"], st["seed"], 0,
                                                    case["shots"], p=case["p"])
        bits, idx, count = msc.prescreen(_ctx(), st["circ"], off, chan, pauli)
        st["chan"][: chan.numel()].copy_(chan)
        st["pauli"][: pauli.numel()].copy_(pauli)
        st["idx"][:count].copy_(idx)
        return dict(off=off, chan=st["chan"], pauli=st["pauli"], bits=bits, idx=st["idx"],
                    count=count)
    msc.twosite_contract(_ctx(), case["chi"], case["batch"], st["A"], st["B"], st["G"],
                         st["theta"], precision=PRECISION[case["precision"]])
    return st["theta"]


# ---------------------------------------------------------------------------
# what a pass cannot do without

RECORD = 64        # bytes of a per-shot record


def work(case):
    kind = case["kind"]
    if kind == "contract":
        chi, batch = case["chi"], case["batch"]
        return dict(bytes=batch * 16.0 * chi * chi * 4, flops=batch * (32.0 * chi ** 3 + 128.0 * chi ** 2))
    _, _, M, flops = CIRCUITS[case["circuit"]]
    n, p = case["shots"], case["p"]
    if kind == "screen":
        csr = 8.0 * (n + 1) + 5.0 * n * M * p
        return dict(bytes=2 * csr + n / 8 + 8.0 * n * 0.2, flops=0.0)
    # the share of a full run that a simulated shot does (measured): with
    # checkpoints a shot starts at its first fault, and a rejecting
    # measurement stops it
    if kind == "batch":
        alive = math.exp(-0.78 * M * p)        # left by the screen
        sims = n if case["space_time"] else alive * n
        share = min(0.5, 0.036 * M * p) if case["prefix"] else 1.0
        return dict(bytes=8.0 * WMAX * 7, flops=sims * share * flops)
    w = case["w_max"] / 2 if case["w_max"] >= 0 else M * p
    sims = case["survivors"] or n
    share = min(0.5, 0.09 * w) if case["prefix"] else 1.0 / (1.0 + 0.5 * w)
    return dict(bytes=8.0 * sims + 5.0 * w * sims + RECORD * sims, flops=sims * share * flops)


# ---------------------------------------------------------------------------
# the same results in double precision, from the state vector

_S = math.sqrt(0.5)
_ONE = {"H": [[_S, _S], [_S, -_S]], "S": [[1, 0], [0, 1j]], "SDG": [[1, 0], [0, -1j]],
        "T": [[1, 0], [0, complex(_S, _S)]], "TDG": [[1, 0], [0, complex(_S, -_S)]],
        "X": [[0, 1], [1, 0]], "Y": [[0, -1j], [1j, 0]], "Z": [[1, 0], [0, -1]]}


def _pauli_rows(psi, rows, q, code):
    """The Pauli with bits (x, z) = code on qubit q of the states `rows`."""
    if code & 3 == 0:
        return
    n = psi.shape[1].bit_length() - 1
    v = psi[rows].view(len(rows), 1 << q, 2, 1 << (n - 1 - q))
    v0, v1 = v[:, :, 0], v[:, :, 1]
    if code & 3 == 1:
        v = torch.stack([v1, v0], dim=2)
    elif code & 3 == 2:
        v = torch.stack([v0, -v1], dim=2)
    else:
        v = torch.stack([-1j * v1, 1j * v0], dim=2)
    psi[rows] = v.reshape(len(rows), -1)


def _state_vector(text, off, chan, pauli, tau_rej=1e-6):
    """(P_acc, fidelity of the seed qubit with the target; 1 if rejected) of
    the shots, by applying every op of the text to full state vectors."""
    dev, S = "cuda", len(off) - 1
    shot_of = np.repeat(np.arange(S), np.diff(off))
    ops, n, seedq, target = [], 0, 0, "T"
    for ln in text.splitlines():
        t = ln.split()
        if not t or t[0] in ("TICK", "SEGMENT", "ORDER") or t[0].startswith("#"):
            continue
        if t[0] == "QUBITS":
            n = int(t[1])
        elif t[0] == "SEED":
            seedq = int(t[1])
        elif t[0] == "TARGET":
            target = t[1]
        else:
            ops.append((t[0], [int(x) for x in t[1:]]))
    psi = torch.zeros(S, 1 << n, dtype=torch.complex128, device=dev)
    psi[:, 0] = 1.0
    p_acc = torch.ones(S, dtype=torch.float64, device=dev)
    alive = torch.ones(S, dtype=torch.bool, device=dev)
    ch = 0

    def slices(qubits, bits):
        """psi with the qubits fixed to the bits, as a view."""
        v = psi.view(S, *([2] * n))
        ix = [slice(None)] * (n + 1)
        for q, b in zip(qubits, bits):
            ix[q + 1] = b
        return v[tuple(ix)]

    for op, a in ops:
        if op in _ONE:
            m = _ONE[op]
            x0, x1 = slices(a, [0]), slices(a, [1])
            if m[0][1] == 0 and m[1][0] == 0:
                if m[0][0] != 1:
                    x0 *= m[0][0]
                x1 *= m[1][1]
            else:
                y0 = m[0][0] * x0 + m[0][1] * x1
                x1.copy_(m[1][0] * x0 + m[1][1] * x1)
                x0.copy_(y0)
        elif op == "CX":
            x0, x1 = slices(a, [1, 0]), slices(a, [1, 1])
            y = x0.clone()
            x0.copy_(x1)
            x1.copy_(y)
        elif op in ("CZ", "CS", "CSDG", "CCZ"):
            slices(a, [1] * len(a)).mul_({"CZ": -1, "CS": 1j, "CSDG": -1j, "CCZ": -1}[op])
        elif op in ("XERR", "DEP1", "DEP2", "DEP3"):
            at = np.nonzero(chan == ch)[0]
            for code in np.unique(pauli[at]) if len(at) else []:
                rows = torch.from_numpy(shot_of[at[pauli[at] == code]]).to(dev)
                for j, q in enumerate(a):
                    _pauli_rows(psi, rows, q, (int(code) >> (2 * j)) & 3)
            ch += 1
        elif op == "M":
            w = psi.view(S, 1 << a[0], 2, -1)
            prob = (w.real.square() + w.imag.square()).sum(dim=(1, 3))
            pe = prob[:, 0] / prob.sum(dim=1).clamp_min(1e-300)
            alive &= pe >= tau_rej
            p_acc = torch.where(alive, p_acc * pe, torch.zeros_like(p_acc))
            scale = torch.where(alive, prob[:, 0].clamp_min(1e-300).rsqrt(), torch.zeros_like(pe))
            w[:, :, 0] *= scale.view(S, 1, 1)
            w[:, :, 1] = 0
        elif op == "R":
            pass    # the first op on a qubit, or after a measurement with outcome 0
        else:
            raise ValueError(op)
    t = np.array([1, complex(_S, _S) if target == "T" else 1j]) * _S
    w = psi.view(S, 1 << seedq, 2, -1)
    amp = np.conj(t[0]) * w[:, :, 0] + np.conj(t[1]) * w[:, :, 1]
    f = (amp.real.square() + amp.imag.square()).sum(dim=(1, 2))
    f = torch.where(alive, f, torch.ones_like(f))
    return p_acc, f.clamp_max(1.0)


def exact(case, seed):
    if case["kind"] == "contract":
        A, B, G = _tensors(case, seed)
        chi, batch = case["chi"], case["batch"]
        if batch * chi ** 3 > 1e10:
            return None
        g = torch.complex(G.double()[0::2], G.double()[1::2]).view(2, 2, 2, 2)   # [i j i' j']
        out = torch.empty(batch, 2, 2 * chi, 2 * chi, dtype=torch.float64, device="cuda")
        for b in range(batch):
            ar, ai, br, bi = A[b, 0].double(), A[b, 1].double(), B[b, 0].double(), B[b, 1].double()
            s = torch.complex(ar @ br - ai @ bi, ar @ bi + ai @ br).view(chi, 2, 2, chi)
            th = torch.zeros_like(s)
            for i in range(2):
                for j in range(2):
                    for k in range(2):
                        for m in range(2):
                            th[:, i, j] += g[i, j, k, m] * s[:, k, m]
            out[b, 0] = th.real.reshape(2 * chi, 2 * chi)
            out[b, 1] = th.imag.reshape(2 * chi, 2 * chi)
        return out
    # the state vector is within reach at 17 qubits and a thousand shots
    if case["kind"] not in ("shots", "camps") or case["circuit"] not in ("7q", "17q"):
        return None
    if case["shots"] > (1 << 16 if case["circuit"] == "7q" else 1500):
        return None
    off, chan, pauli = _faults(case, seed)
    text = _text(case["circuit"])
    sel = np.arange(len(off) - 1)
    if case["survivors"]:
        return None     # which shots are selected is the screen's answer
    p, f = [], []
    step = 4096 if case["circuit"] == "7q" else 128
    for s in range(0, len(sel), step):
        e = min(len(sel), s + step)
        a, b = off[s], off[e]
        x, y = _state_vector(text, off[s:e + 1] - a, chan[a:b], pauli[a:b])
        p.append(x)
        f.append(y)
    return dict(p_acc=torch.cat(p), fidelity=torch.cat(f), chi_peak=None, status=None,
                rejected_at=None, fail=None, n2q=None, flops=None)
