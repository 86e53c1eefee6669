"""Work counted for gates that one launch decomposes whole (up to 64 columns)."""
import numpy as np
import pytest

from paper_2601_04422_amd import workloads as W

pytestmark = pytest.mark.gpu


def test_small_gates_count_their_work():
    """A merge of two sites (8 m chi n and the gate's 32 m n flops), a dot product of
    every pair of columns per sweep (8 flops a row), and the rotations (32 a row):
    at least one each of the m (m - 1) / 2 pairs of a random matrix in the first
    sweep, at most one in every sweep but the last."""
    from paper_2601_04422_amd import tnsim as T

    n, chi = 12, 16
    m = T.MPS(n, chi, 0.0)
    m.import_state(*W.random_canonical_mps(n, W.saturated_dims(n, chi), 4, profile="flat"))
    m.profile(True)
    assert m.apply_2q(5, 6, W.haar_u4(np.random.default_rng(2))) == T.OK
    got, sweeps = m.profile_read()["eig"]["flops"], m.stats()["last_sweeps"]
    c = 2 * chi
    pairs, merge = c * (c - 1) // 2, 8 * c * chi * c + 32 * c * c
    dots = 8 * c * pairs * sweeps
    assert merge + dots + 32 * c * pairs <= got <= merge + dots + 32 * c * pairs * (sweeps - 1)
    m.profile(True)  # clears the totals
    assert m.profile_read()["eig"]["flops"] == 0
