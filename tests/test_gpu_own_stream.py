"""Work on a stream of the caller's own (non-blocking, not ordered with the
default stream) against the same work on the default stream."""
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


def test_gradient(T):
    """One segment of Haar gates to a bond of 64 and rotations: its adjoints run
    on while the host is at the end of tnsim_backward.  The adjoint's sums over
    workgroups are added in any order, so two runs agree to rounding: entries
    are sums of at most 2^14 products of unit vectors."""
    import torch

    n, rng = 14, np.random.default_rng(40)
    gates, param, axis = [], [], []
    for _ in range(2):
        for q in range(n):
            gates.append((q, -1, np.eye(2)))
            param.append(len(axis))
            axis.append(1)
        for layer in W.brickwork_haar(n, 7, int(rng.integers(1 << 30))):
            gates += layer
            param += [-1] * len(layer)
    angles = rng.uniform(0, 2 * np.pi, len(axis))
    paulis = ["I" * i + "ZZ" + "I" * (n - 2 - i) for i in range(n - 1)]
    got = []
    for stream in (None, torch.cuda.Stream(), torch.cuda.Stream()):
        m = T.MPS(n, 64, 0.0, stream=stream)
        loss = m.forward_checkpointed(gates, param, axis, angles, [0], paulis, [1.0] * (n - 1))
        got.append((loss, m.backward(0.7)))
        del m  # the workspace with it
    assert np.max(np.abs(got[0][1])) > 1e-3
    for loss, grad in got[1:]:
        assert abs(loss - got[0][0]) < 1e-12
        assert np.max(np.abs(grad - got[0][1])) < 2.0 ** -53 * 2 ** 14


def _state(T, n, chi, seed, **kw):
    m = T.MPS(n, chi, 0.0, **kw)
    m.import_state(*W.random_canonical_mps(n, W.saturated_dims(n, chi), seed))
    return m


@pytest.mark.parametrize("precision,storage,qr", [("fp64", "c128", False), ("fp64", "c128", True),
                                                  ("bf16x6", "c64", True)])
def test_layers_of_block_gates(T, precision, storage, qr):
    """Bonds of 2 to 100: gates of one workgroup and gates of two to eight
    column blocks in one batch, which converge at different sweeps, so that the
    sweep's graph is replaced while one of its replays is in flight.  The
    captured launches are the eager ones: equal bit for bit."""
    import torch

    n, kw = 20, dict(precision=precision, storage=storage, svd_precondition=qr)
    e = _state(T, n, 100, 5, **kw)
    own = _state(T, n, 100, 5, stream=torch.cuda.Stream(), **kw)
    for layer in W.brickwork_haar(n, 4, 6):
        assert e.apply_layer(layer) == T.OK and own.apply_layer(layer) == T.OK
        rec = e.last_batch()
        block = rec[np.minimum(rec[:, 1], rec[:, 3]) > 32]
        assert len(block) >= 3 and block[:, 5].min() >= 2  # swept, not decomposed in one launch
        assert np.array_equal(rec, own.last_batch())
    assert len(set(rec[:, 5])) > 1
    for q in range(n):
        assert np.array_equal(own.site(q), e.site(q))
    for b in range(n - 1):
        assert np.array_equal(own.lam(b), e.lam(b))


def test_batch_of_handles_with_block_gates(T):
    """Handles of uneven sizes in shared launches on a stream of their own
    against each one by itself.  Another K-split adds a Gram's rows in another
    order: equal to rounding."""
    import torch

    sizes = [(20, 100), (14, 70), (17, 40), (9, 100)]
    s = torch.cuda.Stream()
    own = [_state(T, n, chi, 7 + n, stream=s, max_layer_gates=(40 if k == 0 else 0))
           for k, (n, chi) in enumerate(sizes)]
    alone = [_state(T, n, chi, 7 + n) for n, chi in sizes]
    circuits = [W.brickwork_haar(n, 3, 50 + n) for n, _ in sizes]
    for l in range(3):
        assert T.apply_layer_multi(own, [c[l] for c in circuits]) == T.OK
        for m, c in zip(alone, circuits):
            assert m.apply_layer(c[l]) == T.OK
    for (n, chi), a, b in zip(sizes, alone, own):
        assert list(a.bond_dims()) == list(b.bond_dims())
        for k in range(n - 1):
            assert np.max(np.abs(a.lam(k) - b.lam(k))) < 1e-12
        c = T.MPS(n, chi)
        c.copy_from(b)  # to the stream of `a`
        assert abs(1 - abs(a.overlap(c)) ** 2 / (a.norm2() * c.norm2())) < 1e-12
