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
