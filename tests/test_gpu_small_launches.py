"""One-qubit layers whose descriptors travel as kernel arguments, and reads of
states around the size up to which a kernel moves them to the host."""
import numpy as np
import pytest

from paper_2601_04422_amd import workloads as W

pytestmark = pytest.mark.gpu


def state(T, dims, storage="c128", **kw):
    n = len(dims) - 1
    sites, lams = W.random_canonical_mps(n, dims, 11)
    m = T.MPS(n, max(dims), 0.0, storage=storage,
              precision="fp64" if storage == "c128" else "f32acc", **kw)
    m.import_state(sites, lams)
    return m, sites, lams


@pytest.mark.parametrize("storage", ["c128", "c64"])
@pytest.mark.parametrize("count", [1, 2, 31, 32, 33, 64, 128, 129, 140])
def test_1q_layer_equals_single_gates(count, storage):
    """A layer of `count` gates (whole and partial launches, and the staged
    path above 128) leaves the bits that one call per gate leaves."""
    from paper_2601_04422_amd import tnsim as T

    n = 140
    dims = [1] + [2 + (q % 3) * (1 < q < n - 1) for q in range(1, n)] + [1]
    a, sites, _ = state(T, dims, storage, max_layer_gates=1)
    b = T.MPS(n, max(dims), 0.0, storage=storage, precision=a.precision, max_layer_gates=1)
    b.copy_from(a)
    rng = np.random.default_rng(count)
    gates = []
    for q in rng.permutation(n)[:count]:
        u = np.linalg.qr(rng.normal(size=(2, 2)) + 1j * rng.normal(size=(2, 2)))[0]
        gates.append((int(q), -1, u))
    assert a.apply_layer(gates) == T.OK
    for q, _, u in gates:
        b.apply_1q(q, u)
    eps = 2.0 ** -53 if storage == "c128" else 2.0 ** -24
    for q in range(n):
        assert (a.site(q) == b.site(q)).all()
    for q, _, u in gates:  # four rounded products and their sums, the site rounded twice
        want = np.einsum("st,atb->asb", u, sites[q])
        bound = 8 * eps * np.einsum("st,atb->asb", abs(u), abs(sites[q]))
        assert (abs(a.site(q) - want) <= bound).all()


@pytest.mark.parametrize("storage, width", [("c128", 1), ("c64", 2)])
@pytest.mark.parametrize("right", [1, 15, 16, 17, 64])
def test_reads_return_the_state(right, storage, width):
    """Sites of 16 KB and just below and above, and far above; every bond."""
    from paper_2601_04422_amd import tnsim as T

    n, left = 14, 32 * width
    up = left.bit_length()
    dims = [2 ** q for q in range(up)] + [min(right, 2 ** (n - q)) for q in range(up, n + 1)]
    m, sites, lams = state(T, dims, storage)
    for q, s in enumerate(sites):
        want = s if storage == "c128" else s.astype(np.complex64).astype(np.complex128)
        assert (m.site(q) == want).all()
    for b, l in enumerate(lams):
        assert (m.lam(b) == l).all()
