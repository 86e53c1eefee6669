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


# (chi, preconditioned, weights, sweeps that the order of all column pairs takes)
CAPS = [(12, True, "smooth", 6), (24, True, "flat", 7), (60, False, "smooth", 7),
        (100, True, "smooth", 6)]


@pytest.mark.parametrize("path", ["gate", "layer", "circuit"])
@pytest.mark.parametrize("chi,qr,profile,cap", CAPS)
def test_a_cap_that_the_order_of_all_pairs_meets_is_enough(T, chi, qr, profile, cap, path):
    """Other orders of the rotations, and the one-workgroup SVD without the QR
    preconditioner, need a sweep or more above `cap` here; the gate then starts
    again in the order of all pairs.  One sweep less is refused, sites untouched."""
    n = 16
    q = n // 2 - 1
    sites, lams = W.random_canonical_mps(n, W.saturated_dims(n, chi), 3, profile=profile)
    gates = [(q, q + 1, W.haar_u4(np.random.default_rng(1)))]

    def run(sweeps):
        m = T.MPS(n, chi, 0.0, svd_precondition=qr, jacobi_max_sweeps=sweeps)
        m.import_state(sites, lams)
        st = {"gate": lambda: m.apply_2q(*gates[0]), "layer": lambda: m.apply_layer(gates),
              "circuit": lambda: m.apply_circuit(gates)}[path]()
        return m, st

    ref, st = run(0)
    assert st == T.OK
    m, st = run(cap)
    assert st == T.OK and m.stats()["last_sweeps"] == cap
    assert list(m.last_batch()[:, 5]) == [cap]
    assert np.max(np.abs(m.lam(q) - ref.lam(q))) < 1e-12
    m, st = run(cap - 1)
    assert st == T.E_NOCONV
    assert np.array_equal(m.site(q), sites[q]) and np.array_equal(m.site(q + 1), sites[q + 1])


def test_circuit_goes_on_after_a_second_attempt(T):
    """A circuit on a preconditioned handle whose gates partly exceed the cap at
    the first attempt: the same state as without a cap."""
    n, chi = 14, 100
    layers = W.brickwork_haar(n, 10, 31)
    gates = [g for l in layers for g in l]
    free = T.MPS(n, chi, 1e-12, svd_precondition=True)
    free.run_circuit(gates)
    top = int(free.last_batch()[:, 5].max())
    m = T.MPS(n, chi, 1e-12, svd_precondition=True, jacobi_max_sweeps=top - 1)
    m.run_circuit(gates)
    rec = m.last_batch()
    assert len(rec) == len(gates) and rec[:, 5].max() <= top - 1
    assert list(m.bond_dims()) == list(free.bond_dims())
    assert abs(1 - abs(m.overlap(free)) ** 2 / (m.norm2() * free.norm2())) < 1e-12
