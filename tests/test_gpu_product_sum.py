"""The density as one sum of products (csrc/k_sum.hip): edges of its tiles and the sizes where they
change, short contractions, and the orders that do not take it.

sum_n |c_n| n^2 eps bounds D's error as for the other product forms: order 80, 80^2 * 2.2e-16 * 3 =
4.3e-12; the tests ask for 5e-12.
"""
import numpy as np
import pytest

import synth
from refcheck import density

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

BETA = 4.0


@pytest.fixture(scope="module")
def cd():
    import paper_2306_12616_amd as m

    return m


# 32-tiles to 560, 48-tiles to 700 (32-tiles where the padding ends before the last one, 625..640), ranges of
# 96-tiles, chains from 1345; order 8 has three blocks, order 72 = 9 * 8 no T_72 in its ladder
@pytest.mark.parametrize("n,order", [(16, 80), (17, 8), (32, 80), (33, 80), (64, 8), (129, 80), (559, 80), (560, 80),
                                     (561, 80), (624, 80), (625, 80), (700, 80), (701, 80), (701, 8), (768, 80), (769, 80),
                                     (865, 80), (1008, 80), (1009, 80), (1152, 80), (1153, 80), (1344, 80),
                                     (1344, 8), (1345, 80), (300, 72), (300, 73)])
def test_mu_search_and_density(cd, n, order):
    print(f"product sum n={n} order={order}", flush=True)
    h, q, lam = synth.hamiltonian(n, "uniform", seed=n)
    H = torch.from_numpy(h).cuda()
    handle = cd.Handle(0)
    D = torch.full((n, n + 3), 7.0, dtype=torch.float64, device="cuda")   # odd rows: unaligned output
    for _ in range(3):   # launched, captured, replayed
        D[:, :n] = 0.0
        mu, _, info = cd.chebdm_mu_search(handle, H, BETA, n // 2 + 0.25, order, D=D[:, :n])
        ref, _ = density(q, lam, order, BETA, mu, info["emin"], info["emax"], info["n_quad"])
        got = D.cpu().numpy()
        assert np.array_equal(got[:, :n], got[:, :n].T)
        assert np.max(np.abs(got[:, :n] - ref)) <= 5e-12
        assert np.all(got[:, n:] == 7.0)
    mu1, D1, info1 = cd.chebdm_mu_search(handle, H, BETA, n // 2 + 0.25, order, cd.make_opts(giant="one_chain"))
    assert mu1 == mu and info1["n_gemm"] == info["n_gemm"]
    assert np.max(np.abs(D1.cpu().numpy() - got[:, :n])) <= 1e-11
    handle.close()
