"""Loss and gradient of Pauli sums whose terms have every kind of support (none,
one site at either end, neighbours, ends only, the whole chain, overlapping)
against parameter shifts of a dense state vector; no truncation."""
import numpy as np
import pytest

from paper_2601_04422_amd import workloads as W

pytestmark = pytest.mark.gpu

SUMS = {
    "identity": [("IIIIII", 1.5), ("IIIIII", -0.5)],
    "ends": [("ZIIIII", 0.7), ("IIIIIX", -1.1)],
    "whole": [("XYZXYZ", 1.0)],
    "mixed": [("IIIIII", 0.3), ("IZZIII", 1.0), ("IIXYII", -0.8), ("YIIIIY", 0.6), ("IIIZII", 2.0),
              ("XYZXYZ", -0.4), ("ZZIIII", 1.2), ("IIIIZZ", 0.9)],
}


def dense(n, gates):
    psi = np.zeros((2,) * n, dtype=np.complex128)
    psi[(0,) * n] = 1.0
    for q0, q1, m in gates:
        if q1 < 0:
            psi = np.moveaxis(np.tensordot(m, psi, (1, q0)), 0, q0)
        else:
            psi = np.moveaxis(np.tensordot(m.reshape(2, 2, 2, 2), psi, ((2, 3), (q0, q1))), (0, 1),
                              (q0, q1))
    return psi


def value(n, gates, terms):
    psi = dense(n, gates)
    tot = 0.0
    for p, c in terms:
        phi = psi
        for q, s in enumerate(p):
            phi = np.moveaxis(np.tensordot(W.PAULI[s], phi, (1, q)), 0, q)
        tot += c * np.vdot(psi, phi).real
    return tot


@pytest.mark.parametrize("storage", ["c128", "c64"])
@pytest.mark.parametrize("name", sorted(SUMS))
def test_against_parameter_shift(name, storage):
    from paper_2601_04422_amd import tnsim as T

    n, terms = 6, SUMS[name]
    rng = np.random.default_rng(12)
    rots = [(q, ax) for _ in range(2) for q in range(n) for ax in (1, 2)]
    angles = rng.uniform(0, 2 * np.pi, len(rots))
    half = len(rots) // 2
    u = [W.haar_u4(rng) for _ in range(2 * (n - 1))]
    order, k = [], 0
    for l in range(2):
        order += [("r", i) for i in range(l * half, (l + 1) * half)]
        order += [("g", (j, u[l * (n - 1) + j])) for j in range(n - 1)]

    def circuit(a):
        return [(rots[x][0], -1, W.rot("XYZ"[rots[x][1]], a[x])) if kind == "r"
                else (x[0], x[0] + 1, x[1]) for kind, x in order]

    m = T.MPS(n, 8, 0.0, storage=storage)
    gates = [(q0, q1, g) for q0, q1, g in circuit(np.zeros(len(rots)))]
    param = [x if kind == "r" else -1 for kind, x in order]
    loss = m.forward_checkpointed(gates, param, [ax for _, ax in rots], angles,
                                  [0, len(order) // 2], [p for p, _ in terms],
                                  [c for _, c in terms])
    grad = m.backward(2.0)
    shift = np.zeros(len(rots))
    for i in range(len(rots)):
        for sgn in (1, -1):
            a = angles.copy()
            a[i] += sgn * np.pi / 2
            shift[i] += sgn * value(n, circuit(a), terms)  # (f+ - f-) / 2, times dloss = 2
    weight = sum(abs(c) for _, c in terms)
    # rounding of about 40 gates of at most 16 x 16, in the precision the sites
    # are stored in; the SVD's adjoint divides by gaps of squared singular
    # values (1e-2 allowed for each of two factors)
    eps = 2.0 ** -53 if storage == "c128" else 2.0 ** -24
    assert abs(loss - value(n, circuit(angles), terms)) <= 64 * 40 * eps * weight
    assert np.abs(grad - shift).max() <= min(1e4 * 64 * 40 * eps, 1e-2) * weight
