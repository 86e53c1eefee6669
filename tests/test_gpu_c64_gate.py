"""One two-qubit gate on complex64 sites against numpy's float64 SVD, with and
without the QR preconditioner, at the row counts where its panel kernels
change (256, 512, 1024 rows) and at one and two column blocks."""
import numpy as np
import pytest

from paper_2601_04422_amd import workloads as W

pytestmark = pytest.mark.gpu
EPS32 = 2.0 ** -24


@pytest.mark.parametrize("precondition", [False, True])
@pytest.mark.parametrize("chi", [5, 16, 33, 64, 127, 128, 129, 256, 257, 512, 513])
def test_gate_vs_numpy(chi, precondition):
    from paper_2601_04422_amd import tnsim as T

    n = 2 * int(np.ceil(np.log2(chi))) + 2
    sites, lams = W.random_canonical_mps(n, W.saturated_dims(n, chi), 500 + chi)
    g = W.haar_u4(np.random.default_rng(chi))
    i = n // 2 - 1
    m = T.MPS(n, chi, 0.0, precision="f32acc", storage="c64", svd_precondition=precondition,
              max_layer_gates=1)
    m.import_state(sites, lams)
    assert m.apply_2q(i, i + 1, g) == T.OK
    a, b = (s.astype(np.complex64).astype(np.complex128) for s in sites[i:i + 2])

    def theta(a, b, g):
        t = (a.reshape(-1, a.shape[2]) @ b.reshape(b.shape[0], -1)).reshape(a.shape[0], 4, -1)
        return ((g @ t).reshape(2 * a.shape[0], 2, -1) * lams[i + 1]).reshape(2 * a.shape[0], -1)

    s = np.linalg.svd(theta(a, b, g), compute_uv=False)
    k = min(chi, s.size)
    norm = np.sqrt(np.sum(s[:k] ** 2))
    # sums of chi and of 4 complex products in float32, and the factors rounded
    # once: every entry of theta is off by at most (2 chi + 16) 2^-24 of the
    # same sums over absolute values, a singular value by the norm of that
    err = (2 * chi + 16) * EPS32 * np.linalg.norm(theta(abs(a), abs(b), abs(g))) / norm
    lam = m.lam(i)
    assert lam.size == k
    assert np.abs(lam - s[:k] / norm).max() <= err
    # orthonormal but for the rounding of the stored columns: two factors
    # 2^-24 of sum |u| |u'| <= 1, and as much again for the float64 SVD
    u = m.site(i).reshape(-1, k)
    assert np.abs(u.conj().T @ u - np.eye(k)).max() <= 4 * EPS32
