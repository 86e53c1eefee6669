"""The work that is timed: what users of this framework run, through its public entry points.

A case is a dict of plain values; its ``kind`` says which program it is:

* ``circuit``   a whole small circuit from |0...0>, layer by layer (state-vector sizes);
* ``gate``      one two-qubit gate on a state in hand, the per-gate float64 path;
* ``layer``     one layer (rotations on every qubit, then CNOTs; or Haar gates) on a saturated
                state, all gates batched, then an observable;
* ``batch``     one layer of many independent circuits of uneven sizes in shared launches;
* ``program``   OpenQASM text parsed, fused and run by the dependency scheduler, with gates
                on distant qubits;
* ``gradient``  loss and gradient of a parametrised ansatz (forward and backward);
* ``sample``    shots from a state;
* ``readout``   Pauli expectations, an overlap and amplitudes;
* ``canonical`` a state in a random gauge brought to canonical form.

Gate application works in place, so a pass copies the prepared state into a working handle
first, as a program does that branches from a common prefix.  Site tensors are defined up to a
choice of basis on every bond; outputs are what is not: the Schmidt values of every bond, the
truncation statistics, the state vector of a small circuit, the joined pair of sites of a single
gate, and the norm and an expectation value of larger states.
"""
import math

import numpy as np
import torch

from paper_2601_04422_amd import tnsim as T

I2 = np.eye(2, dtype=np.complex128)
PX = np.array([[0, 1], [1, 0]], dtype=np.complex128)
PY = np.array([[0, -1j], [1j, 0]], dtype=np.complex128)
PZ = np.array([[1, 0], [0, -1]], dtype=np.complex128)
PAULI = {"I": I2, "X": PX, "Y": PY, "Z": PZ}
CNOT = np.array([[1, 0, 0, 0], [0, 1, 0, 0], [0, 0, 0, 1], [0, 0, 1, 0]], dtype=np.complex128)
SWAP = np.array([[1, 0, 0, 0], [0, 0, 1, 0], [0, 1, 0, 0], [0, 0, 0, 1]], dtype=np.complex128)
EPS = 2.0 ** -53


def listed():
    return [
        # the smallest circuits (10 qubits, 10 brickwork layers, no truncation): every call is
        # latency and launches
        {"name": "circuit-n10", "kind": "circuit", "n": 10, "depth": 10, "chi": 32},
        # one gate per call with the constructor's defaults, small and middling odd bonds
        {"name": "gate-chi24", "kind": "gate", "chi": 24, "qr": False},
        {"name": "gate-chi300", "kind": "gate", "chi": 300, "qr": False},
        # layers of the rx/rz + CNOT circuit at the size of the multi-layer checks, and at the
        # largest bond dimension, batched float64 on a stream of its own
        {"name": "layer-chi128", "kind": "layer", "n": 40, "chi": 128, "gates": "rxrz_cnot",
         "cutoff": 1e-12, "precision": "fp64", "storage": "c128"},
        {"name": "layer-chi1024", "kind": "layer", "n": 36, "chi": 1024, "gates": "rxrz_cnot",
         "cutoff": 1e-12, "precision": "fp64", "storage": "c128"},
        # Haar brickwork at n = 64, chi 256, complex64 sites and float32 products
        {"name": "wide-chi256", "kind": "layer", "n": 64, "chi": 256, "gates": "haar",
         "cutoff": 1e-10, "precision": "f32acc", "storage": "c64"},
        # one step of a batch of uneven circuits (split-bf16 products, complex64 sites)
        {"name": "batch-uneven", "kind": "batch", "circuits": 16, "chi": 128},
        # a Trotter program with some distant gates, from text to the scheduler
        {"name": "program-n20", "kind": "program", "n": 20, "steps": 4, "chi": 64},
        # loss and gradient of the Ry/Rz + CNOT-ladder ansatz
        {"name": "gradient-n14", "kind": "gradient", "n": 14, "layers": 4, "chi": 64},
        # a thousand shots from a state in hand
        {"name": "sample-chi256", "kind": "sample", "n": 48, "chi": 256, "shots": 1000},
        # observables, an overlap and amplitudes of a larger state
        {"name": "readout-chi500", "kind": "readout", "n": 28, "chi": 500},
        # canonical form of a state in a random gauge
        {"name": "canonical-chi90", "kind": "canonical", "n": 20, "chi": 90, "qr": True},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["circuit", "gate", "layer", "layer", "batch", "program", "gradient",
                       "sample", "readout", "canonical"])
    if kind == "circuit":
        return {"kind": kind, "n": rng.randint(3, 14), "depth": rng.randint(2, 14),
                "chi": rng.choice([8, 16, 32, 100])}
    if kind == "gate":
        return {"kind": kind, "chi": _log_int(rng, 2, 400), "qr": rng.random() < 0.4}
    if kind == "layer":
        chi = _log_int(rng, 6, 900)
        ramp = 2 * math.ceil(math.log2(chi))
        room = max(2, min(70 - ramp, int(16 * (1024 / chi) ** 2.2)))
        precision, storage = rng.choice([("fp64", "c128"), ("fp64", "c128"), ("f32acc", "c64"),
                                         ("bf16x6", "c64"), ("bf16x3", "c64")])
        return {"kind": kind, "n": ramp + rng.randint(2, room), "chi": chi,
                "gates": rng.choice(["rxrz_cnot", "haar"]),
                "cutoff": rng.choice([0.0, 1e-12, 1e-10]) if storage == "c128" else 1e-10,
                "precision": precision, "storage": storage}
    if kind == "batch":
        return {"kind": kind, "circuits": rng.randint(2, 24), "chi": rng.choice([32, 64, 128, 256])}
    if kind == "program":
        return {"kind": kind, "n": rng.randint(5, 28), "steps": rng.randint(1, 5),
                "chi": rng.choice([32, 64, 96])}
    if kind == "gradient":
        return {"kind": kind, "n": rng.randint(4, 16), "layers": rng.randint(1, 5), "chi": 64}
    if kind == "sample":
        return {"kind": kind, "n": rng.randint(24, 60), "chi": _log_int(rng, 20, 500),
                "shots": _log_int(rng, 10, 4000)}
    if kind == "readout":
        return {"kind": kind, "n": rng.randint(22, 40), "chi": _log_int(rng, 20, 700)}
    return {"kind": kind, "n": rng.randint(10, 24), "chi": _log_int(rng, 8, 110),
            "qr": rng.random() < 0.5}


# ---------------------------------------------------------------- inputs


def _rot(axis, t):
    return math.cos(t / 2) * I2 - 1j * math.sin(t / 2) * PAULI[axis]


def _haar(rng, d):
    z = rng.standard_normal((d, d)) + 1j * rng.standard_normal((d, d))
    q, r = np.linalg.qr(z)
    p = np.diag(r)
    return q * (p / np.abs(p))[None, :]


def _isometry(rng, rows, cols):
    """rows x cols with orthonormal columns and entries spread like a random unitary's: random
    phases between unitary Fourier transforms (quick to make at 2048 x 1024)."""
    if rows <= 64:
        return np.ascontiguousarray(_haar(rng, rows)[:, :cols])
    ph = np.exp(2j * np.pi * rng.random((3, rows)))
    jk = (np.arange(cols)[:, None] * np.arange(rows)[None, :]) % rows
    x = torch.from_numpy(np.exp(-2j * np.pi * np.arange(rows) / rows)[jk] / math.sqrt(rows))
    for k in range(2):
        x = torch.fft.fft(x * torch.from_numpy(ph[k]), norm="ortho")
    return (x * torch.from_numpy(ph[2])).T.contiguous().numpy()


def _weights(rng, chi):
    """A random state's Schmidt spectrum (quarter-circle law), decreasing, squares summing to 1."""
    out = np.empty(0)
    while out.size < chi:
        x = rng.uniform(0.0, 2.0, 2 * chi + 8)
        y = rng.uniform(0.0, 2.0, 2 * chi + 8)
        out = np.concatenate([out, x[x * x + y * y <= 4.0]])
    lam = np.sort(out[:chi])[::-1]
    return lam / np.linalg.norm(lam)


def _dims(n, chi):
    return [min(chi, 2 ** min(q, n - q, 30)) for q in range(n + 1)]


def _state(rng, n, chi, storage="c128"):
    """A left-canonical state whose bonds are as large as chi allows."""
    d = _dims(n, chi)
    sites = [_isometry(rng, 2 * d[q], d[q + 1]).reshape(d[q], 2, d[q + 1]) for q in range(n)]
    if storage == "c64":
        sites = [s.astype(np.complex64).astype(np.complex128) for s in sites]
    return sites, [_weights(rng, d[q + 1]) for q in range(n - 1)]


def _brickwork(rng, n, parity):
    return [(j, j + 1, _haar(rng, 4)) for j in range(parity, n - 1, 2)]


def _layers(rng, case, n):
    parity = int(rng.integers(0, 2)) if n > 2 else 0
    if case["gates"] == "haar":
        return [_brickwork(rng, n, parity)]
    a, b = rng.uniform(0, 2 * math.pi, (2, n))
    return [[(q, -1, _rot("X", a[q])) for q in range(n)],
            [(q, -1, _rot("Z", b[q])) for q in range(n)],
            [(j, j + 1, CNOT) for j in range(parity, n - 1, 2)]]


def _pauli(rng, n, weight=3):
    s = ["I"] * n
    for q in rng.choice(n, min(weight, n), replace=False):
        s[q] = "XYZ"[int(rng.integers(0, 3))]
    return "".join(s)


def _batch_sizes(rng, case):
    sizes = []
    for _ in range(case["circuits"]):
        chi = int(rng.choice([c for c in (32, 64, 128, 256) if c <= case["chi"]]))
        sizes.append((int(rng.integers(16, 41)), chi))
    return sizes


def _program(rng, case):
    """Trotter steps of a Heisenberg chain with fields and one distant cx a step; returns the
    OpenQASM text and the same circuit with the three gates of a bond multiplied."""
    n, dt = case["n"], 0.1
    h = rng.uniform(-1.0, 1.0, n)
    text = ["OPENQASM 2.0;", 'include "qelib1.inc";', f"qreg q[{n}];"]
    gates = []
    for q in range(1, n, 2):
        text.append(f"x q[{q}];")
        gates.append((q, -1, PX))
    bond = np.eye(4, dtype=np.complex128)
    for p in (PX, PY, PZ):
        bond = bond @ (math.cos(dt) * np.eye(4) - 1j * math.sin(dt) * np.kron(p, p))
    for _ in range(case["steps"]):
        for start in (0, 1):
            for j in range(start, n - 1, 2):
                text += [f"{g}({2 * dt!r}) q[{j}],q[{j + 1}];" for g in ("rxx", "ryy", "rzz")]
                gates.append((j, j + 1, bond))
        for q in range(n):
            t = float(2 * dt * h[q])
            text.append(f"rz({t!r}) q[{q}];")
            gates.append((q, -1, _rot("Z", t)))
        d = int(rng.integers(2, min(6, n)))
        a = int(rng.integers(0, n - d))
        c, t = (a, a + d) if rng.random() < 0.5 else (a + d, a)
        text.append(f"cx q[{c}],q[{t}];")
        gates.append((c, t, CNOT))
    return "\n".join(text) + "\n", gates


def _ansatz(rng, case):
    """Ry, Rz on every qubit then the CNOT ladder, per layer; loss sum Z_i Z_i+1."""
    n, gates, param, axis, seg = case["n"], [], [], [], []
    for _ in range(case["layers"]):
        seg.append(len(gates))
        for q in range(n):
            for ax in (1, 2):
                gates.append((q, -1, I2))
                param.append(len(axis))
                axis.append(ax)
        for j in range(n - 1):
            gates.append((j, j + 1, CNOT))
            param.append(-1)
    paulis = ["I" * i + "ZZ" + "I" * (n - 2 - i) for i in range(n - 1)]
    angles = rng.uniform(0, 2 * math.pi, len(axis))
    return gates, param, axis, angles, seg, paulis, [1.0] * (n - 1)


def _random_gauge(rng, sites):
    sites = list(sites)
    for b in range(len(sites) - 1):
        d = sites[b].shape[2]
        g = rng.standard_normal((d, d)) + 1j * rng.standard_normal((d, d))
        x = np.eye(d) + 0.3 * g / math.sqrt(d)
        sites[b] = np.einsum("asb,bc->asc", sites[b], x)
        sites[b + 1] = np.einsum("ab,bsc->asc", np.linalg.inv(x), sites[b + 1])
    return sites


def _inputs(case, seed):
    """Everything a pass depends on, on the host, from the seed alone."""
    rng = np.random.default_rng(seed)
    kind, inp = case["kind"], {}
    if kind == "circuit":
        n = case["n"]
        inp["layers"] = [_brickwork(rng, n, l % 2) for l in range(case["depth"])]
        inp["layers"] = [l for l in inp["layers"] if l]
    elif kind == "gate":
        n = 2 * math.ceil(math.log2(case["chi"])) + 4
        inp["state"] = _state(rng, n, case["chi"])
        q = n // 2 - 1
        pair = (q, q + 1) if rng.random() < 0.5 else (q + 1, q)
        inp["gate"] = (*pair, _haar(rng, 4))
        inp["pauli"] = _pauli(rng, n)
    elif kind == "layer":
        inp["state"] = _state(rng, case["n"], case["chi"], case["storage"])
        inp["layers"] = _layers(rng, case, case["n"])
        inp["pauli"] = _pauli(rng, case["n"])
    elif kind == "batch":
        inp["sizes"] = _batch_sizes(np.random.default_rng(case["circuits"]), case)
        inp["states"] = [_state(rng, n, chi, "c64") for n, chi in inp["sizes"]]
        inp["layers"] = [_brickwork(rng, n, int(rng.integers(0, 2))) for n, _ in inp["sizes"]]
    elif kind == "program":
        inp["text"], inp["gates"] = _program(rng, case)
        inp["pauli"] = _pauli(rng, case["n"], 2).replace("X", "Z").replace("Y", "Z")
    elif kind == "gradient":
        inp["ansatz"] = _ansatz(rng, case)
    elif kind == "sample":
        inp["state"] = _state(rng, case["n"], case["chi"])
        inp["u"] = rng.random((case["shots"], case["n"]))
    elif kind == "readout":
        inp["state"] = _state(rng, case["n"], case["chi"])
        inp["other"] = _state(rng, case["n"], case["chi"])
        inp["paulis"] = [_pauli(rng, case["n"], w) for w in (1, 2, 4)]
        inp["bits"] = rng.integers(0, 2, (4, case["n"])).astype(np.uint8)
    else:
        sites, lams = _state(rng, case["n"], case["chi"])
        inp["state"] = (_random_gauge(rng, sites), lams)
        inp["chi"] = case["chi"]
        inp["pauli"] = _pauli(rng, case["n"])
    return inp


# ---------------------------------------------------------------- a pass


def _mps(n, chi, cutoff=0.0, state=None, **kw):
    m = T.MPS(n, chi, cutoff, **kw)
    if state is not None:
        m.import_state(*state)
    return m


def prepare(case, seed):
    inp = _inputs(case, seed)
    kind, st = case["kind"], {"case": case}
    chi = case["chi"]
    if kind == "circuit":
        st["mps"] = _mps(case["n"], chi)
        st["layers"] = inp["layers"]
    elif kind == "gate":
        n = len(inp["state"][0])
        kw = dict(svd_precondition=case["qr"], max_layer_gates=1)
        st["base"] = _mps(n, chi, 1e-12, inp["state"], **kw)
        st["mps"] = _mps(n, chi, 1e-12, **kw)
        st.update(gate=inp["gate"], pauli=inp["pauli"])
    elif kind == "layer":
        kw = dict(precision=case["precision"], storage=case["storage"], svd_precondition=True,
                  stream=torch.cuda.Stream())
        st["base"] = _mps(case["n"], chi, case["cutoff"], inp["state"], max_layer_gates=1, **kw)
        st["mps"] = _mps(case["n"], chi, case["cutoff"], **kw)
        st.update(layers=inp["layers"], pauli=inp["pauli"])
    elif kind == "batch":
        kw = dict(precision="bf16x6", storage="c64")
        total = sum(len(l) for l in inp["layers"])
        st["base"] = [_mps(n, c, 1e-10, s, max_layer_gates=1, **kw)
                      for (n, c), s in zip(inp["sizes"], inp["states"])]
        st["mps"] = [_mps(n, c, 1e-10, max_layer_gates=max(total, n // 2) if k == 0 else 0, **kw)
                     for k, (n, c) in enumerate(inp["sizes"])]
        st["layers"] = inp["layers"]
    elif kind == "program":
        st["mps"] = _mps(case["n"], chi, 1e-10, svd_precondition=True,
                         stream=torch.cuda.Stream())
        st.update(text=inp["text"], pauli=inp["pauli"])
    elif kind == "gradient":
        st["mps"] = _mps(case["n"], chi)
        st["ansatz"] = inp["ansatz"]
    elif kind == "sample":
        st["mps"] = _mps(case["n"], chi, 0.0, inp["state"], max_layer_gates=1)
        st["u"] = torch.as_tensor(inp["u"], device="cuda:0")
    elif kind == "readout":
        st["mps"] = _mps(case["n"], chi, 0.0, inp["state"], max_layer_gates=1)
        st["other"] = _mps(case["n"], chi, 0.0, inp["other"], max_layer_gates=1)
        st.update(paulis=inp["paulis"], bits=inp["bits"])
    else:
        kw = dict(svd_precondition=case["qr"], max_layer_gates=1)
        st["base"] = _mps(case["n"], chi, 0.0, inp["state"], **kw)
        st["mps"] = _mps(case["n"], chi, 0.0, **kw)
        st["pauli"] = inp["pauli"]
    return st


def _ok(status):
    if status != T.OK:
        raise RuntimeError(f"status {status}")


def _table(lams, n, chi):
    """The Schmidt values of all bonds in one array, every bond with room for its largest rank."""
    d = _dims(n, chi)
    out = np.zeros(sum(d[1:n]))
    for b, l in enumerate(lams):
        at = sum(d[1:b + 1])
        out[at:at + l.size] = l
    return out


def _spectra(m):
    return _table([m.lam(b) for b in range(m.n - 1)], m.n, m.chi_max)


def _vector(m):
    """The state vector of a small state, qubit 0 first."""
    v = np.ones((1, 1), dtype=np.complex128)
    for q in range(m.n):
        a = m.site(q)
        v = (v @ a.reshape(a.shape[0], -1)).reshape(-1, a.shape[2])
    return v[:, 0]


def _pair(m, q):
    """Sites q and q + 1 joined (the basis on the bond between them drops out)."""
    a, b = (torch.from_numpy(m.site(k)).to("cuda:0") for k in (q, q + 1))
    return a.reshape(-1, a.shape[2]) @ b.reshape(b.shape[0], -1)


def _stats(m):
    s = m.stats()
    return np.array([s["sum_eps"], s["prod_keep"]])


def _values(m, pauli):
    """The norm and an observable: two numbers on the scale of the norm."""
    return np.array([m.norm2(), m.expect(pauli)])


def run(st):
    kind, m = st["case"]["kind"], st["mps"]
    if kind == "circuit":
        m.reset()
        m.run_layers(st["layers"])
        return {"lam": _spectra(m), "psi": _vector(m)}
    if kind == "gate":
        m.copy_from(st["base"])
        _ok(m.apply_2q(*st["gate"]))
        q = min(st["gate"][:2])
        return {"lam": m.lam(q), "theta": _pair(m, q), "stats": _stats(m), "value": _values(m, st["pauli"])}
    if kind == "layer":
        m.copy_from(st["base"])
        m.run_layers(st["layers"])
        return {"lam": _spectra(m), "stats": _stats(m), "value": _values(m, st["pauli"])}
    if kind == "batch":
        for a, b in zip(m, st["base"]):
            a.copy_from(b)
        _ok(T.apply_layer_multi(m, st["layers"]))
        return {"lam": np.concatenate([_spectra(a) for a in m]),
                "stats": np.array([_stats(a) for a in m])}
    if kind == "program":
        n, gates = T.parse_qasm(st["text"])
        m.reset()
        m.run_circuit(T.fuse(gates, n))
        return {"lam": _spectra(m), "value": _values(m, st["pauli"])}
    if kind == "gradient":
        loss = m.forward_checkpointed(*st["ansatz"])
        return {"loss": loss, "grad": m.backward(1.0)}
    if kind == "sample":
        bits, logp = m.sample(st["u"])
        return {"bits": bits, "logp": logp}
    if kind == "readout":
        return {"values": np.array([m.expect(p) for p in st["paulis"]]),
                "overlap": np.array([m.norm2(), m.overlap(st["other"])]),
                "amp": np.array([m.amplitude(b) for b in st["bits"]])}
    m.copy_from(st["base"])
    m.canonicalize()
    return {"lam": _spectra(m), "value": _values(m, st["pauli"])}


# ---------------------------------------------------------------- the work of a pass


def _gate_work(cl, cm, cr, k, elem=16):
    """Merge, gate, SVD with left vectors (R-bidiagonalisation count, complex = 4 real), write-back;
    both sites read and written once."""
    m, n = 2 * cl, 2 * cr
    a, b = max(m, n), min(m, n)
    fl = 8.0 * m * cm * n + 32.0 * m * n + 4.0 * (6.0 * a * b * b + 11.0 * b ** 3) + 8.0 * k * m * n
    return fl, elem * (m * cm + cm * n + m * k + k * n)


def _layer_work(n, chi, bonds, elem):
    d = _dims(n, chi)
    w = [_gate_work(d[j], d[j + 1], d[j + 2], d[j + 1], elem) for j in bonds]
    return sum(x[0] for x in w), sum(x[1] for x in w)


def work(case):
    kind, chi = case["kind"], case["chi"]
    fl = by = 0.0
    if kind == "circuit":
        for l in range(case["depth"]):
            f, b = _layer_work(case["n"], min(chi, 2 ** (l + 1)), range(l % 2, case["n"] - 1, 2), 16)
            fl, by = fl + f, by + b
    elif kind == "gate":
        fl, by = _gate_work(chi, chi, chi, chi)
    elif kind == "layer":
        elem = 16 if case["storage"] == "c128" else 8
        fl, by = _layer_work(case["n"], chi, range(0, case["n"] - 1, 2), elem)
    elif kind == "batch":
        for n, c in _batch_sizes(np.random.default_rng(case["circuits"]), case):
            f, b = _layer_work(n, c, range(0, n - 1, 2), 8)
            fl, by = fl + f, by + b
    elif kind == "program":
        for s in range(case["steps"]):
            f, b = _layer_work(case["n"], min(chi, 4 ** (s + 1)), range(case["n"] - 1), 16)
            fl, by = fl + f, by + b
    elif kind == "gradient":
        for s in range(case["layers"]):
            f, b = _layer_work(case["n"], min(chi, 2 ** (s + 1)), range(case["n"] - 1), 16)
            fl, by = fl + 4 * f, by + 3 * b
    else:
        n, d = case["n"], _dims(case["n"], chi)
        site = sum(2.0 * d[q] * d[q + 1] for q in range(n))
        pair = sum(8.0 * 2 * d[q] * d[q + 1] * (d[q] + d[q + 1]) for q in range(n))
        if kind == "sample":
            fl = pair + sum(8.0 * 2 * d[q] * d[q + 1] * min(case["shots"], 2 ** min(30, n - q))
                            for q in range(n))
            by = 16 * site + case["shots"] * (9.0 * n + 8)
        elif kind == "readout":  # three expectations and an overlap; amplitudes read half a site
            fl, by = 4 * pair, 16 * (2 * site)
        else:
            fl = 2 * sum(_gate_work(d[q], d[q + 1], d[q + 2], d[q + 1])[0] for q in range(n - 1))
            by = 32 * site
    return {"bytes": float(by), "flops": float(fl)}


# ---------------------------------------------------------------- the same in 64 bits on the host


class _Ref:
    """Plain numpy MPS: left-canonical sites, Schmidt weights, gates by full SVD."""

    def __init__(self, n, chi, cutoff, state=None):
        self.n, self.chi, self.cutoff = n, chi, cutoff
        if state is None:
            self.a = [np.array([1.0, 0.0], dtype=np.complex128).reshape(1, 2, 1) for _ in range(n)]
            self.lam = [np.ones(1) for _ in range(n - 1)]
        else:
            self.a, self.lam = [s.copy() for s in state[0]], [l.copy() for l in state[1]]
        self.sum_eps, self.keep = 0.0, 1.0

    def gate(self, q0, q1, g):
        if q1 < 0:
            self.a[q0] = np.einsum("st,atb->asb", g, self.a[q0])
            return
        lo, hi = min(q0, q1), max(q0, q1)
        if hi - lo > 1:
            for j in range(hi - 1, lo, -1):
                self.gate(j, j + 1, SWAP)
            self.gate(*((lo, lo + 1) if q0 == lo else (lo + 1, lo)), g)
            for j in range(lo + 1, hi):
                self.gate(j, j + 1, SWAP)
            return
        if q0 > q1:
            g = SWAP @ g @ SWAP
        al, ar = self.a[lo], self.a[hi]
        cl, cr = al.shape[0], ar.shape[2]
        th = (al.reshape(2 * cl, -1) @ ar.reshape(ar.shape[0], -1)).reshape(cl, 4, cr)
        th = (g @ th).reshape(2 * cl, 2, cr)
        w = self.lam[lo + 1] if lo + 1 < self.n - 1 else np.ones(1)
        u, s, _ = np.linalg.svd((th * w).reshape(2 * cl, 2 * cr), full_matrices=False)
        s2 = s * s
        tail = np.concatenate([np.cumsum(s2[::-1])[::-1], [0.0]])
        k = next(k for k in range(1, s.size + 1) if k == s.size or tail[k] <= self.cutoff * tail[0])
        k = max(1, min(k, self.chi, int(np.sum(s2 > 2 * cl * EPS * s2[0]))))
        norm = math.sqrt(np.sum(s2[:k]))
        self.sum_eps += tail[k] / tail[0]
        self.keep *= 1.0 - tail[k] / tail[0]
        self.a[lo] = u[:, :k].reshape(cl, 2, k)
        self.a[hi] = (u[:, :k].conj().T @ th.reshape(2 * cl, 2 * cr)).reshape(k, 2, cr) / norm
        self.lam[lo] = s[:k] / norm

    def stats(self):
        return np.array([self.sum_eps, self.keep])


def _contract(bra, ket, pauli=None):
    e = np.ones((1, 1), dtype=np.complex128)
    for q, (b, k) in enumerate(zip(bra, ket)):
        f = (e @ k.reshape(k.shape[0], -1)).reshape(b.shape[0], 2, k.shape[2])
        if pauli and pauli[q] != "I":
            f = np.einsum("st,atb->asb", PAULI[pauli[q]], f)
        e = b.reshape(-1, b.shape[2]).conj().T @ f.reshape(-1, k.shape[2])
    return complex(e[0, 0])


def _expect(a, pauli):
    return _contract(a, a, pauli) / _contract(a, a).real


def _ref_values(a, pauli):
    return np.array([_contract(a, a).real, _expect(a, pauli)])


def _amp(a, bits):
    v = np.ones((1, 1), dtype=np.complex128)
    for s, b in zip(a, bits):
        v = v @ s[:, int(b), :]
    return complex(v[0, 0])


def _svd_flops(case):
    return work(case)["flops"]


def _exact_gradient(inp, n):
    gates, param, axis, angles, _, _, _ = inp["ansatz"]
    th = torch.tensor(angles, dtype=torch.float64, requires_grad=True)
    psi = torch.zeros((2,) * n, dtype=torch.complex128)
    psi[(0,) * n] = 1.0
    for (q0, q1, _), p in zip(gates, param):
        if p >= 0:
            psi = psi.reshape(2 ** q0, 2, -1)
            c, s = torch.cos(th[p] / 2), torch.sin(th[p] / 2)
            if axis[p] == 1:
                psi = torch.stack([c * psi[:, 0] - s * psi[:, 1], s * psi[:, 0] + c * psi[:, 1]], 1)
            else:
                ph = torch.complex(c, s)
                psi = torch.stack([ph.conj() * psi[:, 0], ph * psi[:, 1]], 1)
        else:
            psi = psi.reshape(2 ** q0, 2, 2, -1)
            psi = torch.stack([psi[:, 0], psi[:, 1].flip(1)], 1)
    prob = (psi.real ** 2 + psi.imag ** 2).reshape(-1)
    idx = torch.arange(2 ** n)
    z = torch.zeros(2 ** n, dtype=torch.float64)
    for i in range(n - 1):
        z += 1.0 - 2.0 * (((idx >> i) ^ (idx >> (i + 1))) & 1).double()
    loss = (prob * z).sum()
    loss.backward()
    return {"loss": float(loss.detach()), "grad": th.grad.numpy()}


def _exact_sample(inp):
    sites, u = inp["state"][0], inp["u"]
    env = [np.ones((1, 1), dtype=np.complex128)]
    for a in sites[:-1]:
        f = np.tensordot(env[-1], a, 1)
        env.append(np.tensordot(a.conj(), f, ((0, 1), (0, 1))))
    shots, n = u.shape
    v = np.ones((shots, 1), dtype=np.complex128)
    bits, logp = np.zeros((shots, n), dtype=np.uint8), np.zeros(shots)
    for q in range(n - 1, -1, -1):
        w = [v @ sites[q][:, s, :].T for s in (0, 1)]
        p = [np.sum((x.conj() @ env[q]) * x, 1).real for x in w]
        one = u[:, q] >= p[0] / (p[0] + p[1])
        bits[:, q] = one
        pr = np.where(one, p[1], p[0])
        logp += np.log(pr / (p[0] + p[1]))
        v = np.where(one[:, None], w[1], w[0]) / np.sqrt(pr)[:, None]
    return {"bits": torch.from_numpy(bits), "logp": torch.from_numpy(logp)}


def _exact_canonical(inp):
    a = list(inp["state"][0])
    n = len(a)
    for q in range(n - 1):
        x, r = np.linalg.qr(a[q].reshape(-1, a[q].shape[2]))
        a[q] = x.reshape(a[q].shape[0], 2, -1)
        a[q + 1] = np.tensordot(r, a[q + 1], 1)
    a[-1] = a[-1] / np.linalg.norm(a[-1])
    value, lam = _ref_values(a, inp["pauli"]), [None] * (n - 1)
    for q in range(n - 1, 0, -1):
        u, s, v = np.linalg.svd(a[q].reshape(a[q].shape[0], -1), full_matrices=False)
        k = int(np.sum(s * s > EPS * 2 * a[q - 1].shape[0] * s[0] ** 2))
        lam[q - 1] = s[:k] / np.linalg.norm(s[:k])
        a[q] = v[:k].reshape(k, 2, -1)
        a[q - 1] = np.tensordot(a[q - 1], u[:, :k] * s[:k], 1)
    return {"lam": _table(lam, n, inp["chi"]), "value": value}


def exact(case, seed):
    kind = case["kind"]
    if kind in ("gate", "layer", "batch", "program", "canonical") and _svd_flops(case) > 3e11:
        return None
    inp = _inputs(case, seed)
    if kind == "circuit":
        r = _Ref(case["n"], case["chi"], 0.0)
        for layer in inp["layers"]:
            for g in layer:
                r.gate(*g)
        v = np.ones((1, 1), dtype=np.complex128)
        for a in r.a:
            v = (v @ a.reshape(a.shape[0], -1)).reshape(-1, a.shape[2])
        return {"lam": _table(r.lam, r.n, r.chi), "psi": v[:, 0]}
    if kind == "gate":
        r = _Ref(len(inp["state"][0]), case["chi"], 1e-12, inp["state"])
        r.gate(*inp["gate"])
        q = min(inp["gate"][:2])
        a, b = r.a[q], r.a[q + 1]
        return {"lam": r.lam[q], "stats": r.stats(),
                "theta": torch.from_numpy(a.reshape(-1, a.shape[2]) @ b.reshape(b.shape[0], -1)),
                "value": _ref_values(r.a, inp["pauli"])}
    if kind == "layer":
        r = _Ref(case["n"], case["chi"], case["cutoff"], inp["state"])
        for layer in inp["layers"]:
            for g in layer:
                r.gate(*g)
        return {"lam": _table(r.lam, r.n, r.chi), "stats": r.stats(), "value": _ref_values(r.a, inp["pauli"])}
    if kind == "batch":
        refs = []
        for (n, chi), state, layer in zip(inp["sizes"], inp["states"], inp["layers"]):
            refs.append(_Ref(n, chi, 1e-10, state))
            for g in layer:
                refs[-1].gate(*g)
        return {"lam": np.concatenate([_table(r.lam, r.n, r.chi) for r in refs]),
                "stats": np.array([r.stats() for r in refs])}
    if kind == "program":
        r = _Ref(case["n"], case["chi"], 1e-10)
        for g in inp["gates"]:
            r.gate(*g)
        return {"lam": _table(r.lam, r.n, r.chi), "value": _ref_values(r.a, inp["pauli"])}
    if kind == "gradient":
        return _exact_gradient(inp, case["n"])
    if kind == "sample":
        return _exact_sample(inp)
    if kind == "readout":
        a, b = inp["state"][0], inp["other"][0]
        return {"values": np.array([_expect(a, p) for p in inp["paulis"]]),
                "overlap": np.array([_contract(a, a).real, _contract(a, b)]),
                "amp": np.array([_amp(a, x) for x in inp["bits"]])}
    return _exact_canonical(inp)
