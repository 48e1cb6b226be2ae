"""Trace moments where the Gram pass splits its matrices: sizes around the 16-wide diagonal blocks (a
single block, a last block of one row, whole blocks) and 1, 2 and 3 groups of 16 matrices a side."""
import numpy as np
import pytest

import synth
from oracle import chebyshev as ch

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def cd():
    import paper_2306_12616_amd as m

    return m


@pytest.fixture(scope="module")
def handle(cd):
    h = cd.Handle(0)
    yield h
    h.close()


@pytest.mark.parametrize("n", [1, 2, 15, 16, 17, 31, 32, 33, 127, 128, 129, 640, 1009])
@pytest.mark.parametrize("order", [5, 60, 400, 1300])
def test_moments(cd, handle, n, order):
    if n == 1:
        h = np.array([[0.3]])
    else:
        h, _, _ = synth.hamiltonian(n, "uniform", seed=n)
    lam = np.linalg.eigvalsh(h)
    tau = cd.chebdm_moments(handle, torch.from_numpy(h).cuda(), order, cd.make_opts(), -1.3, 1.2 + abs(lam).max())
    ref = ch.moments_from_eigs(lam, -1.3, 1.2 + abs(lam).max(), order)
    # rounding of T_j grows like j^2 and adds over the n diagonal entries
    assert np.max(np.abs(tau - ref)) <= 4 * order ** 2 * n * np.finfo(float).eps
