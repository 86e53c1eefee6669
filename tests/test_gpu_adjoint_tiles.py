"""Gradients at bond dimensions on both sides of the adjoint products' tile
sizes (matrices of 4 to 128 rows and columns; no truncation), against parameter
shifts of a dense state vector."""
import numpy as np
import pytest

from paper_2601_04422_amd import workloads as W
from test_gpu_adjoint_terms import value

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("storage", ["c128", "c64"])
@pytest.mark.parametrize("n, chi", [(4, 4), (7, 8), (10, 32), (11, 33), (12, 64), (13, 64)])
def test_gradient(n, chi, storage):
    from paper_2601_04422_amd import tnsim as T

    rng = np.random.default_rng(n)
    angles = rng.uniform(0, 2 * np.pi, 3)
    at = [(0, 1), (n // 2, 2), (n - 1, 1)]  # first, middle and last qubit; Y, Z, Y
    depth = int(np.ceil(n / 2)) + 1         # every bond full before the last rotations
    walls = [[(j, j + 1, W.haar_u4(rng)) for j in range(l % 2, n - 1, 2)] for l in range(depth)]

    def circuit(a):
        gates, par = [], []
        for l, wall in enumerate(walls):
            if l == depth - 2:
                for k, (q, ax) in enumerate(at):
                    gates.append((q, -1, W.rot("XYZ"[ax], a[k])))
                    par.append(k)
            gates += wall
            par += [-1] * len(wall)
        return gates, par

    terms = [("I" * (n // 2 - 1) + "XZ" + "I" * (n - n // 2 - 1), 1.0), ("Z" + "I" * (n - 1), -0.5)]
    gates, par = circuit(angles)
    m = T.MPS(n, chi, 0.0, storage=storage)
    loss = m.forward_checkpointed(gates, par, [ax for _, ax in at], angles, [0, len(gates) // 2],
                                  [p for p, _ in terms], [c for _, c in terms])
    grad = m.backward(1.0)
    # rounding of the gates (64 of it allowed each, for sums of up to 128 terms)
    # in the precision the sites are stored in; the SVD's adjoint divides by gaps
    # of squared singular values (1e-2 allowed for each of two factors)
    eps = 2.0 ** -53 if storage == "c128" else 2.0 ** -24
    weight = sum(abs(c) for _, c in terms)
    tol = 64 * len(gates) * eps * weight
    assert abs(loss - value(n, gates, terms)) <= tol
    for k in range(3):
        shift = np.zeros(3)
        shift[k] = np.pi / 2
        want = (value(n, circuit(angles + shift)[0], terms)
                - value(n, circuit(angles - shift)[0], terms)) / 2
        assert abs(grad[k] - want) <= min(1e4 * tol, 1e-2 * weight)
