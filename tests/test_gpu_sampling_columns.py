"""Draws of very many shots at once, whose products take tiles of their own, against
the same draws a few hundred at a time."""
import numpy as np
import pytest

from paper_2601_04422_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("storage", ["c128", "c64"])
@pytest.mark.parametrize("chi,shots", [(13, 3000), (33, 9000), (100, 20000), (129, 20011)])
def test_all_at_once_equals_in_parts(chi, shots, storage):
    """Bonds of 1 to chi (K of every kind, ragged tiles, columns gathered for bits 0
    and 1).  The same sums in another order: log-probabilities to n chi roundings
    of conditionals, the strings equal (no uniform lies that close to one)."""
    from paper_2601_04422_amd import tnsim as T

    n = 16
    m = T.MPS(n, chi, 0.0, storage=storage)
    m.import_state(*W.random_canonical_mps(n, W.saturated_dims(n, chi), chi))
    u = np.random.default_rng(shots).random((shots, n))
    bits, logp = m.sample(u)
    part = [m.sample(u[k:k + 311]) for k in range(0, shots, 311)]
    assert np.array_equal(bits.cpu().numpy(), np.concatenate([b.cpu().numpy() for b, _ in part]))
    want = np.concatenate([l.cpu().numpy() for _, l in part])
    assert np.max(np.abs(logp.cpu().numpy() - want)) < 1e-11
