"""The loss of a Pauli sum at bonds where its environments' products change
kernels (64) against the expectation values of the same state, which are
contracted term by term."""
import numpy as np
import pytest

from paper_2601_04422_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("storage", ["c128", "c64"])
@pytest.mark.parametrize("chi", [63, 64, 100])
def test_loss_equals_expectations(chi, storage):
    """Terms of every support.  Both sides add products of unit vectors, at most
    2 chi of them an entry, through 14 sites: equal to 14 x 2 chi roundings."""
    from paper_2601_04422_amd import tnsim as T

    n, rng = 14, np.random.default_rng(chi)
    gates = [g for l in W.brickwork_haar(n, 9, 7) for g in l] + [(6, -1, np.eye(2))]
    param = [-1] * (len(gates) - 1) + [0]
    terms = ["I" * n, "".join("XYZ"[k] for k in rng.integers(0, 3, n)), "Z" + "I" * (n - 2) + "X",
             "I" * 6 + "ZZ" + "I" * 6, "IIIIXYIZIIIIII", "I" * (n - 1) + "Y", "X" + "I" * (n - 1)]
    coeffs = rng.uniform(-1, 1, len(terms))
    m = T.MPS(n, chi, 0.0, storage=storage)
    loss = m.forward_checkpointed(gates, param, [1], [0.4], [0], terms, coeffs)
    assert max(m.bond_dims()) == chi
    want = sum(c * m.expect(p).real for c, p in zip(coeffs, terms))
    assert abs(loss - want) < 2.0 ** -53 * n * 2 * chi * np.abs(coeffs).sum()
