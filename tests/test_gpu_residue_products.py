"""Float64 products by residue arithmetic (csrc/k_rns.hip) at the sizes where they can go wrong.

Low orders keep the runs short: order 30 takes 10 products (T_2..T_6 in stages, five giant steps).
Rounding in T_n grows at most like n^2 machine epsilons, so sum_n |c_n| n^2 eps <= 30^2 * 2.2e-16
* (sum |c_n| < 3) = 6e-13 bounds D's error; the tests ask for 1e-12.
"""
import numpy as np
import pytest

import synth
from oracle import chebyshev as ch
from refcheck import coeffs, density

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

ORDER, BETA = 30, 4.0


@pytest.fixture(scope="module")
def cd():
    import paper_2306_12616_amd as m

    return m


@pytest.fixture(scope="module")
def handle(cd):
    h = cd.Handle(0)
    yield h
    h.close()


# edges of the 128- and 256 x 128 tiles, of the 64-wide K steps, and past the longest sum that one
# reduction step covers (5120)
@pytest.mark.parametrize("n", [1400, 1408, 1409, 1473, 2999, 3000, 3073, 3136, 5121])
def test_density_at_tile_edges(cd, handle, n):
    print(f"residue products n={n}", flush=True)
    h, q, lam = synth.hamiltonian(n, "uniform", seed=n)
    H = torch.from_numpy(h).cuda()
    D = torch.full((n, n + 3), 7.0, dtype=torch.float64, device="cuda")   # odd rows: unaligned output
    d, info = cd.chebdm_density(handle, H, BETA, 0.1, ORDER, D=D[:, :n])
    ref, _ = density(q, lam, ORDER, BETA, 0.1, info["emin"], info["emax"], info["n_quad"])
    got = D.cpu().numpy()
    assert np.array_equal(got[:, :n], got[:, :n].T)
    assert np.max(np.abs(got[:, :n] - ref)) <= 1e-12
    assert np.all(got[:, n:] == 7.0)


def test_row_scales(cd, handle):
    # rows of very different size: zero, squares below the float64 range, ordinary; bounds [-1, 1]
    # make H~ = H, and a diagonal H keeps every product diagonal
    n = 1400
    d = np.random.default_rng(0).uniform(-1.0, 1.0, n)
    d[:6] = [0.0, 1e-160, -1e-200, 1e-300, 1.0, -1.0]
    H = torch.diag(torch.from_numpy(d)).cuda()
    D, info = cd.chebdm_density(handle, H, BETA, 0.1, ORDER, emin=-1.0, emax=1.0)
    got = D.cpu().numpy()
    p = ch.cheb_eval(coeffs(ORDER, BETA, 0.1, -1.0, 1.0, info["n_quad"]), d)
    assert np.max(np.abs(np.diag(got) - p)) <= 1e-12
    assert np.all(got[~np.eye(n, dtype=bool)] == 0.0)


def test_bounds_inside_the_spectrum(cd, handle):
    # T_n grows to about 1e29 outside [-1, 1]: the row scales follow it.  The trace moments are
    # compared: D itself would multiply the coefficients' rounding by the T_n.
    n = 1400
    h, _, lam = synth.hamiltonian(n, "uniform", seed=5)
    tau = cd.chebdm_moments(handle, torch.from_numpy(h).cuda(), ORDER, emin=-0.2, emax=0.2)
    a, b = np.ones(n, dtype=np.longdouble), (lam / 0.2).astype(np.longdouble)
    for t in tau:
        assert abs(t - a.sum()) <= 1e-12 * np.abs(a).sum()
        a, b = b, 2 * (lam / 0.2) * b - a


# where the 256 x 128 tiles begin, and one row, column or K step past their edges
@pytest.mark.parametrize("n", [1535, 1536, 1537, 1663, 1665, 1793])
def test_density_where_large_tiles_begin(cd, handle, n):
    test_density_at_tile_edges(cd, handle, n)


# launches of several products on the int8 units, single ones on the float64 units: the first and last
# sizes of the rule, the gap in it, four chains (order 80: 9 blocks), ladder and blocks in the same slots.
# sum |c_n| n^2 eps <= 80^2 * 2.2e-16 * 3 = 4.3e-12
@pytest.mark.parametrize("n", [959, 960, 1024, 1025, 1057, 1153, 1399, 1400])
@pytest.mark.parametrize("bounds", ["gershgorin", "lanczos"])
def test_mixed_units(cd, handle, n, bounds):
    print(f"mixed units n={n} {bounds}", flush=True)
    order = 80
    h, q, lam = synth.hamiltonian(n, "uniform", seed=n)
    H = torch.from_numpy(h).cuda()
    for _ in range(2):   # the second call replays the first one's launches
        mu, D, info = cd.chebdm_mu_search(handle, H, BETA, n // 2 + 0.5, order, cd.make_opts(bounds=bounds))
        ref, _ = density(q, lam, order, BETA, mu, info["emin"], info["emax"], info["n_quad"])
        assert np.max(np.abs(D.cpu().numpy() - ref)) <= 5e-12


@pytest.mark.parametrize("n", [1400, 1537])
def test_own_bounds_need_no_row_scales(cd, handle, n):
    # bounds computed by the call put every T_n's rows below norm 1, given ones do not: two routes.
    # One site is alone at the middle of the bounds (a zero row in T_1), one at their end.
    h, _, _ = synth.hamiltonian(n, "uniform", seed=8)
    h[3, :] = h[:, 3] = h[9, :] = h[:, 9] = 0.0
    H = torch.from_numpy(h).cuda()
    lo, hi = cd.chebdm_bounds(handle, H)
    h[3, 3], h[9, 9] = 0.5 * (lo + hi), hi
    H = torch.from_numpy(h).cuda()
    own, _ = cd.chebdm_density(handle, H, BETA, 0.1, ORDER)
    given, _ = cd.chebdm_density(handle, H, BETA, 0.1, ORDER, emin=lo, emax=hi)
    assert (own - given).abs().max().item() <= 2e-12
    tau = [cd.chebdm_moments(handle, H, 60, cd.make_opts(), *b) for b in ((np.nan, np.nan), (lo, hi))]
    assert np.max(np.abs(tau[0] - tau[1])) <= 4 * 60 ** 2 * n * np.finfo(float).eps


def test_bounds_as_close_as_their_rounding(cd, handle):
    # half the width is a few ulps of the centre: (e - cen) / half leaves [-1, 1], T_n grows, and the call
    # keeps the row scales that it takes for given bounds
    n = 1400
    H = torch.diag(torch.from_numpy(1.0 + np.arange(n) % 4 * np.finfo(float).eps)).cuda()
    lo, hi = cd.chebdm_bounds(handle, H)
    assert lo < hi
    tau = [cd.chebdm_moments(handle, H, ORDER, cd.make_opts(), *b) for b in ((np.nan, np.nan), (lo, hi))]
    assert np.array_equal(tau[0], tau[1])


def test_non_finite_rows(cd, handle):
    n = 1400
    h, _, _ = synth.hamiltonian(n, "uniform", seed=6)
    for bad in (np.nan, np.inf):
        h[5, 7] = h[7, 5] = bad
        D, _ = cd.chebdm_density(handle, torch.from_numpy(h).cuda(), BETA, 0.1, ORDER, emin=-1.5, emax=1.5)
        got = D.cpu().numpy()
        assert not np.isfinite(got[5]).any() and not np.isfinite(got[:, 7]).any()
