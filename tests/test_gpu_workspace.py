"""A call that fails leaves nothing behind: the next valid call on the same handle or plan has the bits of a
fresh one's.

A search without a bracket has NaN coefficients, and a scalar matrix in a batch a NaN map; both write
the workspace before the status is known.  Sizes with a padding that later reads reach: n not a
multiple of 16 (Gram, float64), of 128 (Gram, reduced forms), odd (residue planes).
"""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

BETA, ORDER = 0.5, 70


@pytest.fixture(scope="module")
def cd():
    import paper_2306_12616_amd as m

    return m


def results(cd, handle, H, n, opts):
    mu, D, _ = cd.chebdm_mu_search(handle, H, BETA, n // 2 + 0.5, ORDER, opts)
    E, _ = cd.chebdm_density(handle, H, BETA, 0.1, ORDER, opts)
    return [np.array(mu), D.cpu().numpy(), E.cpu().numpy(), cd.chebdm_moments(handle, H, ORDER, opts)]


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16x3"])
@pytest.mark.parametrize("giant", ["composition", "one_chain", "four_chains"])
@pytest.mark.parametrize("n", [77, 333, 1401, 1537])
def test_call_after_a_search_without_bracket(cd, prec, giant, n):
    print(f"after a bracket error n={n} {prec} {giant}", flush=True)
    H = torch.from_numpy(synth.hamiltonian(n, "uniform", seed=n)[0]).cuda()
    opts = cd.make_opts(prec=prec, giant=giant)
    fresh, used = cd.Handle(0), cd.Handle(0)
    want = results(cd, fresh, H, n, opts)
    with pytest.raises(cd.ChebdmError, match="expansion"):   # occupations near 1/2 reach n - 1e-3 nowhere
        cd.chebdm_mu_search(used, H, 0.01, n - 1e-3, ORDER, opts)
    for a, b in zip(want, results(cd, used, H, n, opts)):
        assert np.isfinite(a).all() and np.array_equal(a, b)
    fresh.close()
    used.close()


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16x3"])
@pytest.mark.parametrize("spoil", ["bracket", "scalar"])
def test_batch_after_a_failed_problem(cd, prec, spoil):
    sizes = [33, 101, 333, 1001]
    print(f"batch after {spoil} {prec}", flush=True)
    Hs = [torch.from_numpy(synth.hamiltonian(n, "uniform", seed=n)[0]).cuda() for n in sizes]
    betas, n_elecs = [BETA] * len(sizes), [n // 2 + 0.5 for n in sizes]
    out = []
    for bad in (False, True):
        handle = cd.Handle(0)
        plan = cd.chebdm_batch_create(handle, sizes, ORDER, cd.make_opts(prec=prec))
        if bad and spoil == "bracket":
            plan.mu_search(Hs, [0.01] * len(sizes), [n - 1e-3 for n in sizes], allow_errors=True)
        elif bad:
            plan.mu_search([torch.eye(n, dtype=torch.float64, device="cuda") for n in sizes], betas, n_elecs,
                           allow_errors=True)
        mu, Ds, status, _, _ = plan.mu_search(Hs, betas, n_elecs, allow_errors=True)
        out.append([np.array(mu), np.array(status)] + [d.cpu().numpy() for d in Ds])
        plan.close()
        handle.close()
    for a, b in zip(*out):
        assert np.isfinite(a).all() and np.array_equal(a, b)


def test_plan_destroyed_after_its_handle(cd):
    # as when a collector frees both: the plan's destruction has to leave no error for the next launch
    other = cd.Handle(0)
    for _ in range(8):
        handle = cd.Handle(0)
        plan = cd.chebdm_batch_create(handle, [16, 33], 8)
        handle.close()
        plan.close()
        assert np.isfinite(cd.chebdm_coeffs(other, 5.0, 0.1, -1.0, 1.0, 8)).all()
    other.close()
