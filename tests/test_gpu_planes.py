"""Memory of the residue planes (csrc/api.hip): given back when an allocation needs it, fewer of them on a fuller
device, and the largest sizes, where only three operand sets fit and sums take two reductions.
"""
import pytest

import synth
from refcheck import coeffs

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

BETA = 4.0


@pytest.fixture(scope="module")
def cd():
    import paper_2306_12616_amd as m

    return m


def test_planes_go_back_when_an_allocation_fails(cd):
    n, order = 2000, 80
    H = torch.from_numpy(synth.hamiltonian(n, "uniform", seed=n)[0]).cuda()
    handle = cd.Handle(0)
    D = torch.empty_like(H)
    want = []
    for _ in range(3):   # launched, captured, replayed
        mu, _, _ = cd.chebdm_mu_search(handle, H, BETA, n // 2 + 0.5, order, D=D)
        want.append((mu, D.clone()))
    held = torch.cuda.mem_get_info()[0]
    print("a batch plan of 3 TB", flush=True)
    with pytest.raises(cd.ChebdmError, match="cannot allocate"):
        cd.chebdm_batch_create(handle, [65535], 2000)
    assert torch.cuda.mem_get_info()[0] - held >= 12 * 15 * n * n   # the sets at least
    for _ in range(3):
        mu, _, _ = cd.chebdm_mu_search(handle, H, BETA, n // 2 + 0.5, order, D=D)
        want.append((mu, D.clone()))
    for mu, d in want[1:]:
        assert mu == want[0][0] and torch.equal(d, want[0][1])
    handle.close()


def test_planes_leave_memory_to_others(cd):
    # n = 9600 has six sets of 1.40e9 bytes and 0.71e9 of residues, the workspace of order 30 is 8.9e9: with 36e9
    # bytes free four sets fit a quarter of what is left, with 18e9 one, and the float64 units do the products
    n, order = 9600, 30
    H = torch.randn((n, n), dtype=torch.float64, device="cuda", generator=torch.Generator("cuda").manual_seed(n))
    H = H.tril()
    H += H.tril(-1).t().contiguous()
    out = []
    for left in (None, 36e9, 18e9):
        handle = cd.Handle(0)
        torch.cuda.empty_cache()   # before D, which would hold on to the last filler's block
        D = torch.empty_like(H)
        free = torch.cuda.mem_get_info()[0]
        print(f"planes with {left or free} bytes free", flush=True)
        filler = torch.empty(int(free - left) if left else 0, dtype=torch.uint8, device="cuda")
        before = torch.cuda.mem_get_info()[0]
        try:
            cd.chebdm_density(handle, H, 1e-3, 0.1, order, D=D)
            out.append((D, before - torch.cuda.mem_get_info()[0] - 8.95e9))   # bytes of the planes
        finally:
            handle.close()
            del filler
            torch.cuda.empty_cache()
    assert torch.equal(out[0][0], out[1][0]) and (out[0][0] - out[2][0]).abs().max().item() <= 1.2e-12
    assert out[0][1] >= 6 * 1.4e9 and 3 * 1.4e9 <= out[1][1] <= (36e9 - 8.9e9) / 4 and out[2][1] <= 0.3e9


# the last size with three sets and the first without; order 30 has ten products.  H is dense with entries of
# unit variance, D's reference the same polynomial by float64 products.  Rounding in T_n grows at most
# like n^2 machine epsilons: 30^2 * 2.2e-16 * (sum |c_n| < 3) = 6e-13; the reference has as much.
@pytest.mark.parametrize("n", [13760, 13761])
def test_largest_sizes(cd, n):
    order = 30
    print(f"largest sizes n={n}", flush=True)
    H = torch.randn((n, n), dtype=torch.float64, device="cuda", generator=torch.Generator("cuda").manual_seed(n))
    H = H.tril()
    H += H.tril(-1).t().contiguous()
    handle = cd.Handle(0)
    D, info = cd.chebdm_density(handle, H, 1e-3, 0.1, order, cd.make_opts(bounds="lanczos"))
    handle.close()
    lo, hi = info["emin"], info["emax"]
    c = coeffs(order, 1e-3, 0.1, lo, hi, info["n_quad"])
    eye = torch.eye(n, dtype=torch.float64, device="cuda")
    H.sub_(eye, alpha=0.5 * (lo + hi)).div_(0.5 * (hi - lo))
    t0, t1 = eye, H.clone()
    D.sub_(eye, alpha=c[0]).sub_(t1, alpha=c[1])
    for i in range(2, order + 1):
        t0, t1 = t1, torch.addmm(t0, H, t1, beta=-1.0, alpha=2.0)
        D.sub_(t1, alpha=c[i])
    assert D.abs().max().item() <= 1.2e-12
