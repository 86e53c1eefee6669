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


@pytest.mark.parametrize("split", [1, 4, 16])
def test_gram_splits_agree_to_rounding(T, split):
    """Matrices of up to eight column blocks, whose Grams the table splits over
    1, 4 or 16 row chunks (what their rows allow) against the built-in rule."""
    n = 16
    a, b = (T.MPS(n, 100, 0.0) for _ in range(2))
    for m in (a, b):
        m.import_state(*W.random_canonical_mps(n, W.saturated_dims(n, 100), 2))
    a.set_autotune([0] * 4 + [split] * 4)
    a.profile(True)
    for layer in W.brickwork_haar(n, 2, 8):
        assert a.apply_layer(layer) == T.OK and b.apply_layer(layer) == T.OK
    assert a.profile_read()["gram"]["launches"] > 0
    assert list(a.bond_dims()) == list(b.bond_dims())
    for k in range(n - 1):
        assert np.max(np.abs(a.lam(k) - b.lam(k))) < 1e-12


@pytest.mark.parametrize("precision,storage", [("fp64", "c128"), ("bf16x6", "c64")])
def test_launches_of_many_pairs(T, precision, storage):
    """Four handles of 40 gates, up to eight column pairs each: 1056 pairs and
    more than 24576 tiles in a launch, which takes the pair solves that share a CU
    and the rotation by whole tiles, against each handle by itself, which takes
    neither.  One K-split, so every sum has the same order: equal bit for bit
    with complex64 sites; the pair solve by passes is compiled anew for two to a
    CU, which may contract its products otherwise: equal to rounding."""
    n, chi = 80, 256
    kw = dict(precision=precision, storage=storage, svd_precondition=True)
    one = W.random_canonical_mps(16, W.saturated_dims(16, chi), 9)
    rng = np.random.default_rng(10)
    bulk = [W.random_isometry(rng, 2 * chi, chi).reshape(chi, 2, chi) for _ in range(3)]
    sites = one[0][:8] + [bulk[q % 3] for q in range(n - 16)] + one[0][8:]
    lams = one[1][:8] + [one[1][7]] * (n - 16) + one[1][8:]
    circuits = [W.brickwork_haar(n, 1, 20 + k)[0] for k in range(4)]

    def handle(k):
        m = T.MPS(n, chi, 1e-12, max_layer_gates=(160 if k == 0 else 0), **kw)
        m.import_state(sites, lams)
        m.set_autotune([0, 0, 0, 0, 1, 1, 1, 1])
        return m

    batch = [handle(k) for k in range(4)]
    big = sum(1 for q in range(0, n - 1, 2) if min(q, n - 2 - q) >= 8) * 4
    assert big * 8 > 512 and big * 8 * (2 * chi // 16) > 24576
    assert T.apply_layer_multi(batch, circuits) == T.OK
    for k in range(4):
        alone = T.MPS(n, chi, 1e-12, **kw)
        alone.import_state(sites, lams)
        alone.set_autotune([0, 0, 0, 0, 1, 1, 1, 1])
        assert alone.apply_layer(circuits[k]) == T.OK
        if storage == "c64":
            _equal(alone, batch[k])
        else:
            assert list(alone.bond_dims()) == list(batch[k].bond_dims())
            for b in range(n - 1):
                assert np.max(np.abs(alone.lam(b) - batch[k].lam(b))) < 1e-12
            f = abs(alone.overlap(batch[k])) ** 2 / (alone.norm2() * batch[k].norm2())
            assert abs(1 - f) < 1e-12
        alone.close()
