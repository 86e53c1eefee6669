"""The Jacobi SVD at the ends of its range: matrices whose squared Gram entries
overflow, and sweep caps close to what the decomposition takes."""
import numpy as np
import pytest

from paper_2601_04422_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def T():
    import torch

    assert torch.cuda.is_available()
    from paper_2601_04422_amd import tnsim

    return tnsim


def _state(T, n, chi, scale=1.0, **kw):
    sites, lams = W.random_canonical_mps(n, W.saturated_dims(n, chi), 3, profile="flat")
    sites[n // 2 - 1] = sites[n // 2 - 1] * scale
    m = T.MPS(n, chi, 0.0, **kw)
    m.import_state(sites, lams)
    return m, sites


@pytest.mark.parametrize("chi", [16, 60])
def test_overflowing_rotations_do_not_converge(T, chi):
    """Squared column norms of 1e156: their differences squared are infinite.
    No rotation angle comes of that, so the gate is refused and its sites stay."""
    n = 16
    m, sites = _state(T, n, chi, 1e78)
    q = n // 2 - 1
    assert m.apply_2q(q, q + 1, W.haar_u4(np.random.default_rng(1))) == T.E_NOCONV
    assert np.array_equal(m.site(q), sites[q])
    assert np.array_equal(m.site(q + 1), sites[q + 1])
