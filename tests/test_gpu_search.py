"""Coefficients and mu search where their launches change: quadrature sizes of either parity and step
counts around the eight bisection steps of a launch and the 48 of all of them."""
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


# M nodes: the smallest for the order, odd (a node at x = 0), around a work-group's 512 nodes a turn
@pytest.mark.parametrize("order,n_quad", [(0, 1), (0, 2), (3, 4), (4, 5), (31, 32), (32, 33), (63, 513), (64, 1025),
                                          (100, 2048), (500, 4099)])
def test_coefficients_any_quadrature(cd, handle, order, n_quad):
    c = cd.chebdm_coeffs(handle, 5.0, 0.1, -1.2, 1.0, order, n_quad)
    ref = ch.chebyshev_coeffs(order, 5.0 * 1.1, (0.1 + 0.1) / 1.1, n_quad)
    assert np.max(np.abs(c - ref)) <= 2e-15   # sums of n_quad occupations in [0, 1], divided by n_quad


@pytest.mark.parametrize("max_iter", [1, 2, 7, 8, 9, 16, 17, 40, 47, 48, 49, 52])
@pytest.mark.parametrize("n_quad", [0, 301])
def test_bisection_steps(cd, handle, max_iter, n_quad):
    # one step at a time in the oracle, eight a launch on the device: the same points.  Past some 40
    # steps t - N_e is rounding, so there only the distance to the root is compared.
    n, order, beta, ne = 96, 100, 20.0, 40.5
    h, _, lam = synth.hamiltonian(n, "uniform", seed=11)
    mu, _, info = cd.chebdm_mu_search(handle, torch.from_numpy(h).cuda(), beta, ne, order,
                                      cd.make_opts(max_iter=max_iter, tol=1e-300, n_quad=n_quad), want_density=False)
    half, cen = 0.5 * (info["emax"] - info["emin"]), 0.5 * (info["emax"] + info["emin"])
    tau = ch.moments_from_eigs(lam, info["emin"], info["emax"], order)
    ref, it, _, status = ch.bisect_mu(tau, order, beta * half, ne, 1e-300, max_iter, info["n_quad"])
    if max_iter <= 40:
        assert info["iters"] == it == max_iter and info["status"] == status == 1
        assert abs((mu - cen) / half - ref) <= 4e-16
    else:
        assert info["iters"] <= max_iter and abs((mu - cen) / half - ref) <= 2.0 ** -38
