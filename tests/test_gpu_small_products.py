"""Float64 products of small matrices (csrc/k_small.hip): edges of the 32-wide tiles, of the chunks a
wavefront owns and of the sizes and product counts that take this path.

Order 30 takes 10 products in launches of one and two; the same rounding bound as for the residue
products holds (30^2 eps sum |c_n| < 6e-13), so the tests ask for 1e-12.
"""
import pytest

import numpy as np
import synth
from refcheck import density

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

ORDER, BETA = 30, 4.0


@pytest.fixture(scope="module")
def cd():
    import paper_2306_12616_amd as m

    return m


@pytest.mark.parametrize("n", [2, 16, 31, 32, 33, 127, 128, 129, 256, 257, 384, 385, 512, 513, 735, 736, 737])
@pytest.mark.parametrize("giant", ["composition", "power"])
def test_density_small(cd, n, giant):
    print(f"small products n={n} {giant}", flush=True)
    h, q, lam = synth.hamiltonian(n, "uniform", seed=n)
    handle = cd.Handle(0)
    D = torch.full((n, n + 1), 7.0, dtype=torch.float64, device="cuda")
    _, info = cd.chebdm_density(handle, torch.from_numpy(h).cuda(), BETA, 0.1, ORDER, cd.make_opts(giant=giant),
                                D=D[:, :n])
    ref, _ = density(q, lam, ORDER, BETA, 0.1, info["emin"], info["emax"], info["n_quad"])
    got = D.cpu().numpy()
    assert np.array_equal(got[:, :n], got[:, :n].T)
    assert np.max(np.abs(got[:, :n] - ref)) <= (1e-12 if giant == "composition" else 1e-10)
    assert np.all(got[:, n:] == 7.0)
