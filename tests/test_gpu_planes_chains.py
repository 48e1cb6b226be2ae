"""Chains of giant steps where launches of several products go to the int8 units and single ones do not: planes are
reused and forgotten across baby steps, ladder, block sums and chains.  Three calls with one output (launched,
captured, replayed) have the same bits.

sum_n |c_n| n^2 eps bounds D's error as for the other product forms: order 80, 80^2 * 2.2e-16 * 3 = 4.3e-12; the
tests ask for 5e-12.
"""
import numpy as np
import pytest

import synth
from refcheck import density

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

BETA, ORDER = 4.0, 80


@pytest.fixture(scope="module")
def cd():
    import paper_2306_12616_amd as m

    return m


def three_calls(call, D):
    out = []
    for _ in range(3):
        D.fill_(7.0)
        info = call()
        out.append((info, D.cpu().numpy()))
    for info, d in out[1:]:
        assert info == out[0][0] and np.array_equal(d, out[0][1])
    return out[0]


# the first and last sizes of the rule, its gap (1025..1056), chains below and above the sum of products' end, and
# all launches on the int8 units
@pytest.mark.parametrize("n", [960, 1024, 1025, 1057, 1153, 1344, 1399, 1400])
def test_chains_and_replays(cd, n):
    h, q, lam = synth.hamiltonian(n, "uniform", seed=n)
    H = torch.from_numpy(h).cuda()
    handle = cd.Handle(0)
    D = torch.empty_like(H)
    for bounds in ("gershgorin", "lanczos"):
        for giant in ("composition", "one_chain", "two_chains", "four_chains", "power"):
            print(f"chains n={n} {bounds} {giant}", flush=True)
            opts = cd.make_opts(bounds=bounds, giant=giant)
            for kind in ("mu", "density"):
                def call():
                    if kind == "mu":
                        return cd.chebdm_mu_search(handle, H, BETA, n // 2 + 0.5, ORDER, opts, D=D)[2]
                    return cd.chebdm_density(handle, H, BETA, 0.1, ORDER, opts, D=D)[1]
                info, d = three_calls(call, D)
                ref, _ = density(q, lam, ORDER, BETA, info["mu"], info["emin"], info["emax"], info["n_quad"])
                # the power form's coefficients grow like 2^m |c| (m = 9)
                assert np.max(np.abs(d - ref)) <= 5e-12 * (2 ** 9 if giant == "power" else 1)
                assert np.array_equal(d, d.T)
    handle.close()
