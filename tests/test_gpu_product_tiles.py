"""Overlaps, Pauli expectations and sampling against numpy at bond dimensions
around the tile edges of the complex products (32 and 64) and on both sides of
the size where the larger tiles take over."""
import numpy as np
import pytest

from paper_2601_04422_amd import workloads as W

pytestmark = pytest.mark.gpu
PAULI = {"I": np.eye(2), "X": np.array([[0, 1], [1, 0]]), "Y": np.array([[0, -1j], [1j, 0]]),
         "Z": np.diag([1.0, -1.0])}


def contract(bra, ket, pauli=None):
    e = np.ones((1, 1), dtype=np.complex128)
    for q, (b, k) in enumerate(zip(bra, ket)):
        if pauli:
            k = np.einsum("st,atb->asb", PAULI[pauli[q]], k)
        f = (e @ k.reshape(k.shape[0], -1)).reshape(-1, k.shape[2])
        e = b.reshape(-1, b.shape[2]).conj().T @ f
    return complex(e[0, 0])


@pytest.mark.parametrize("storage", ["c128", "c64"])
@pytest.mark.parametrize("chi", [1, 2, 15, 31, 32, 33, 63, 64, 65, 100, 129, 256, 300, 720])
def test_overlap_expect_sample(chi, storage):
    from paper_2601_04422_amd import tnsim as T

    n = 2 * int(np.ceil(np.log2(chi))) + 3 if chi > 1 else 5
    dims = W.saturated_dims(n, chi)
    states = []
    for seed in (1, 2):
        sites, lams = W.random_canonical_mps(n, dims, 40 * chi + seed)
        if storage == "c64":
            sites = [s.astype(np.complex64).astype(np.complex128) for s in sites]
        states.append((sites, lams))
    ms = []
    for sites, lams in states:
        m = T.MPS(n, chi, 0.0, storage=storage, max_layer_gates=1)
        m.import_state(sites, lams)
        ms.append(m)
    a, b = states[0][0], states[1][0]
    # products of unit-norm factors: chi rounding errors a sum, 2 n sums in a row
    tol = 4 * n * chi * 2.0 ** -53
    norm = contract(a, a).real
    assert abs(ms[0].norm2() - norm) <= tol
    assert abs(ms[0].overlap(ms[1]) - contract(a, b)) <= tol
    for q, p in ((0, "X"), (n // 2, "Y"), (n - 1, "Z")):
        s = ["I"] * n
        s[q] = p
        s[n // 2 - 1] = "Z"
        assert abs(ms[0].expect("".join(s)) - contract(a, a, s) / norm) <= 2 * tol
    assert ms[0].expect("I" * n) == pytest.approx(1.0, abs=2.0 ** -51)
    for shots in (1, 70):
        bits, logp = ms[0].sample(np.random.default_rng(chi).random((shots, n)))
        for x, lp in zip(bits.cpu().numpy()[:4], logp.cpu().numpy()):
            v = np.ones((1, 1))
            for s, bit in zip(a, x):
                v = v @ s[:, bit, :]
            # every conditional is a quotient of two sums of chi^2 terms
            assert abs(lp - np.log(abs(v[0, 0]) ** 2 / norm)) <= 64 * tol
