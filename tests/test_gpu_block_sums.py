"""Block sums on and above the diagonal only (csrc/k_combine.hip): what is left below it is never read.

A first call fills the workspace with NaN; the same handle's next call has to give the bits of a fresh
handle.  Sizes: the first of the upper form, edges of its 32-wide blocks, of the 48- and 64-tiles.
"""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

BETA = 20.0


@pytest.fixture(scope="module")
def cd():
    import paper_2306_12616_amd as m

    return m


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16x3", "bf16x6"])
@pytest.mark.parametrize("n", [700, 735, 961, 1153, 1200, 1537])
@pytest.mark.parametrize("giant", ["composition", "one_chain", "two_chains", "four_chains", "power"])
def test_stale_lower_parts(cd, prec, n, giant):
    if giant == "power" and prec != "fp64":
        pytest.skip("the power form is float64 only")
    print(f"block sums n={n} {prec} {giant}", flush=True)
    h, _, _ = synth.hamiltonian(n, "uniform", seed=n)
    H = torch.from_numpy(h).cuda()
    bad = torch.full_like(H, float("nan"))
    opts = cd.make_opts(prec=prec, giant=giant)
    out = []
    for spoil in (False, True):
        handle = cd.Handle(0)
        for order in (8, 70) if n == 700 else (70,):
            for search in (True, False):
                if spoil:
                    cd.chebdm_density(handle, bad, BETA, 0.1, order, opts, emin=-1.5, emax=1.5)
                if search:
                    _, D, _ = cd.chebdm_mu_search(handle, H, BETA, n // 2 + 0.5, order, opts)
                else:
                    D, _ = cd.chebdm_density(handle, H, BETA, 0.1, order, opts)
                out.append(D.cpu().numpy())
        handle.close()
    half = len(out) // 2
    for a, b in zip(out[:half], out[half:]):
        assert np.isfinite(a).all() and np.array_equal(a, a.T)
        assert np.array_equal(a, b)


# rows and tiles of 32, problems smaller than a work-group's share, two blocks (order 8) and many;
# a spoiled plan's next call against a fresh plan's
@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16x3"])
@pytest.mark.parametrize("order", [8, 70, 700])
def test_batch_stale_lower_parts(cd, prec, order):
    sizes = [33, 64, 100, 257, 640, 1000]
    print(f"batched block sums {prec} order={order}", flush=True)
    Hs = [torch.from_numpy(synth.hamiltonian(n, "uniform", seed=n)[0]).cuda() for n in sizes]
    betas, n_elecs = [BETA] * len(sizes), [n // 2 + 0.5 for n in sizes]
    out = []
    for spoil in (False, True):
        handle = cd.Handle(0)
        plan = cd.chebdm_batch_create(handle, sizes, order, cd.make_opts(prec=prec))
        if spoil:
            plan.mu_search([torch.full_like(h, float("nan")) for h in Hs], betas, n_elecs, allow_errors=True)
        for _ in range(2):
            Ds = plan.mu_search(Hs, betas, n_elecs)[1]
            out.append([d.cpu().numpy() for d in Ds])
        plan.close()
        handle.close()
    for a in out:
        for d, e in zip(a, out[0]):
            assert np.isfinite(d).all() and np.array_equal(d, d.T) and np.array_equal(d, e)
