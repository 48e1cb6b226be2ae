"""Float64 calls keep the digits of D's small entries where H has structure: weakly coupled fragments and
rows that are nearly all diagonal, at sizes whose dense matrices take fixed-point products.

For H = H_0 + eps C with H_0 C-free (block diagonal or diagonal) the entries of D where C is are eps sum_n c_n T_n',
T_{n+1}' = 2 (K T_n' + K' T_n) - T_{n-1}', up to a relative eps^2 (fragments) or eps (diagonal).  Rounding in T_n'
grows at most like n^2 eps: 60^2 * 2.2e-16 * (sum |c_n| < 3) = 2.4e-12 of the block's largest entry on
either side; the tests ask for 5e-12.
"""
import numpy as np
import pytest

import synth
from refcheck import coeffs

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

ORDER, BETA = 60, 20.0


@pytest.fixture(scope="module")
def cd():
    import paper_2306_12616_amd as m

    return m


def problem(kind, n):
    """H_0, C (both n x n on the device) and eps."""
    dense = synth.hamiltonian(n, "uniform", seed=n)[0]
    if kind[0] == "diagonal":
        h0 = np.diag(np.random.default_rng(n).uniform(-1.0, 1.0, n))
        c = dense - np.diag(np.diag(dense))
    else:
        part = np.zeros(n, dtype=bool)
        part[np.random.default_rng(n).permutation(n)[:n // 2 if kind[0] == "halves" else 8]] = True
        same = part[:, None] == part[None, :]
        h0, c = np.where(same, dense, 0.0), np.where(same, 0.0, dense)
    return torch.from_numpy(h0).cuda(), torch.from_numpy(c).cuda(), kind[1]


def derivative(h0, c, lo, hi, mu, n_quad):
    """sum_n c_n dT_n((H_0 + eps C - cen) / half) / d eps."""
    coef = coeffs(ORDER, BETA, mu, lo, hi, n_quad)
    eye = torch.eye(h0.shape[0], dtype=torch.float64, device="cuda")
    k, dk = (h0 - 0.5 * (lo + hi) * eye) / (0.5 * (hi - lo)), c / (0.5 * (hi - lo))
    t0, t1, d0, d1 = eye, k, torch.zeros_like(k), dk
    out = coef[1] * d1
    for i in range(2, ORDER + 1):
        t0, t1, d0, d1 = t1, 2 * (k @ t1) - t0, d1, 2 * (k @ d1 + dk @ t1) - d0
        out = out + coef[i] * d1
    return out


@pytest.mark.parametrize("n", [1000, 1400])
@pytest.mark.parametrize("kind", [("halves", 1e-7), ("halves", 1e-10), ("halves", 1e-17), ("eight", 1e-10),
                                  ("diagonal", 1e-13)], ids=str)
def test_small_entries(cd, n, kind):
    h0, c, eps = problem(kind, n)
    H = (h0 + eps * c).contiguous()
    handle = cd.Handle(0)
    lo, hi = cd.chebdm_bounds(handle, H)
    runs = {}
    for bounds in ("gershgorin", "lanczos"):
        opts = cd.make_opts(bounds=bounds, giant="four_chains")
        D, info = cd.chebdm_density(handle, H, BETA, 0.1, ORDER, opts)
        runs["density", bounds] = 0.1, D, info
        runs["mu", bounds] = cd.chebdm_mu_search(handle, H, BETA, n // 2 + 0.5, ORDER, opts)
    D, info = cd.chebdm_density(handle, H, BETA, 0.1, ORDER, emin=lo, emax=hi)
    runs["density", "given"] = 0.1, D, info
    for name, (mu, D, info) in runs.items():
        print(f"small entries n={n} {kind} {name}", flush=True)
        want = derivative(h0, c, info["emin"], info["emax"], mu, info["n_quad"])
        err = torch.where(c != 0.0, D / eps - want, torch.zeros_like(D)).abs().max().item()
        assert err <= 5e-12 * want[c != 0.0].abs().max().item()
    handle.close()
