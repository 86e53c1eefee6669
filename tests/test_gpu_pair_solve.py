"""One two-qubit gate against numpy's SVD at the column counts where the block
Jacobi changes: one, two, three and four pairs of 32-column blocks (padded
and full), and a sweep long enough that the passes inside the blocks are
spread over its rounds."""
import numpy as np
import pytest

from paper_2601_04422_amd import workloads as W

pytestmark = pytest.mark.gpu
EPS = 2.0 ** -53


def reference(sites, lams, i, g):
    """Merged, gated theta' of sites i, i + 1 and its weighted SVD."""
    a, b = sites[i], sites[i + 1]
    th = (a.reshape(-1, a.shape[2]) @ b.reshape(b.shape[0], -1)).reshape(a.shape[0], 4, -1)
    th = (g @ th).reshape(2 * a.shape[0], 2, -1)
    u, s, _ = np.linalg.svd((th * lams[i + 1]).reshape(th.shape[0], -1), full_matrices=False)
    return th.reshape(th.shape[0], -1), u, s


@pytest.mark.parametrize("precondition", [False, True])
@pytest.mark.parametrize("chi, profile", [
    (2, "flat"), (7, "smooth"), (16, "flat"), (31, "flat"), (32, "smooth"), (33, "flat"),
    (64, "flat"), (64, "smooth"), (65, "flat"), (96, "smooth"), (100, "flat"), (309, "flat")])
def test_gate_vs_numpy(chi, profile, precondition):
    from paper_2601_04422_amd import tnsim as T

    n = 2 * int(np.ceil(np.log2(chi))) + 2
    sites, lams = W.random_canonical_mps(n, W.saturated_dims(n, chi), 900 + chi, profile=profile)
    g = W.haar_u4(np.random.default_rng(chi))
    m = T.MPS(n, chi, 0.0, svd_precondition=precondition, max_layer_gates=1)
    m.import_state(sites, lams)
    i = n // 2 - 1
    assert m.apply_2q(i, i + 1, g) == T.OK
    th, u, s = reference(sites, lams, i, g)
    k = min(chi, s.size)
    norm = np.sqrt(np.sum(s[:k] ** 2))
    # the Jacobi tolerance is rows * 2^-53 per column pair, so a singular value
    # moves by at most rows * sqrt(columns) * 2^-53 of the largest; and the
    # kept subspace by that over the gap at the cut
    err = s.size ** 1.5 * EPS * s[0] / norm
    lam = m.lam(i)
    assert lam.size == k
    assert np.abs(lam - s[:k] / norm).max() <= 4 * err
    gap = (s[k - 1] - (s[k] if k < s.size else 0.0)) / norm
    a, b = m.site(i), m.site(i + 1)
    a, b = a.reshape(-1, k), b.reshape(k, -1)
    assert np.abs(a.conj().T @ a - np.eye(k)).max() <= 8 * s.size * EPS
    kept = u[:, :k] @ (u[:, :k].conj().T @ th) / norm
    assert np.abs(a @ b - kept).max() <= (8 * err + 8 * err / gap) * np.abs(kept).max()
