"""The launch table (tnsim_autotune, tnsim_set_launch_table) decides the rows per
rotation workgroup in every class of launches and changes no result; nor do the
kernels that only launches of many pairs take."""
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


def _equal(a, b):
    assert list(a.bond_dims()) == list(b.bond_dims())
    for q in range(a.n):
        assert np.array_equal(a.site(q), b.site(q))
    for k in range(a.n - 1):
        assert np.array_equal(a.lam(k), b.lam(k))


@pytest.mark.parametrize("precision,storage", [("fp64", "c128"), ("bf16x6", "c64")])
def test_rows_of_the_table_are_taken(T, precision, storage):
    """Rotation bytes count each workgroup's read of V (64 x 64 x 16 bytes), so
    they tell the workgroups: rows of 64 to 200 in chunks of 16 or 128."""
    n = 16
    state = W.random_canonical_mps(n, W.saturated_dims(n, 100), 2)
    layer = W.brickwork_haar(n, 2, 8)[1]
    ms, groups = [], []
    for rows in (64, 512):
        m = T.MPS(n, 100, 0.0, precision=precision, storage=storage)
        m.import_state(*state)
        m.set_autotune([rows] * 4 + [1] * 4)
        m.profile(True)
        assert m.apply_layer(layer) == T.OK
        rot = m.profile_read()["rot"]
        rows_done = rot["flops"] / (8 * 64 * 64)
        groups.append((rot["bytes"] - 32 * 64 * rows_done) / (16 * 64 * 64))
        ms.append(m)
    assert groups[0] > 3 * groups[1] > 0
    _equal(*ms)


def test_autotuned_table_is_taken(T):
    n = 16
    a, b = (T.MPS(n, 100, 0.0, precision="bf16x6", storage="c64") for _ in range(2))
    for m in (a, b):
        m.import_state(*W.random_canonical_mps(n, W.saturated_dims(n, 100), 2))
    table = a.autotune()
    a.set_autotune(table[:4] + [1] * 4)
    b.set_autotune([0] * 4 + [1] * 4)
    for layer in W.brickwork_haar(n, 2, 8):
        assert a.apply_layer(layer) == T.OK and b.apply_layer(layer) == T.OK
    _equal(a, b)
