"""Rounding of the Chebyshev coefficients: no more than that of a sum with one rounded cosine a term."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
pytest.importorskip("torch")

ORDER = 512
LD = np.longdouble
PI = LD("3.14159265358979323846264338327950288")


def one_cosine_a_term(f, cosines, q):
    """sum_j f_j cos in float64: 256 strided chains of fused multiply-adds, then a tree; rows: n."""
    acc = np.zeros((q.shape[0], 256))
    for r in range(0, f.size, 256):
        acc = (f[r:r + 256].astype(LD) * cosines[q[:, r:r + 256]].astype(np.float64) + acc).astype(np.float64)
    acc = acc.reshape(-1, 4, 64)
    for off in (32, 16, 8, 4, 2, 1):
        acc = acc + acc[:, :, np.arange(64) ^ off]
    return ((acc[:, 0, 0] + acc[:, 1, 0]) + acc[:, 2, 0]) + acc[:, 3, 0]


def test_no_more_rounding_than_a_cosine_a_term():
    # pooled over (beta', mu~) and 4 <= n <= 512 (c_0 .. c_3 are of order one: single roundings of the result
    # outweigh the sum's).  The errors that matter are those of some twenty coefficients in each of
    # twelve sums, so the ratio of the two root mean squares scatters by about 1 / sqrt(2 * 240) = 5 %; 8 % is
    # allowed.
    import paper_2306_12616_amd as cd

    handle = cd.Handle(0)
    n = np.arange(4, ORDER + 1)
    got, want = [], []
    for m in (8192, 16384):
        j = 2 * np.arange(m, dtype=np.int64) + 1
        cosines = np.cos(PI * np.arange(4 * m).astype(LD) / (2 * m))
        x = cosines[j]
        for beta, mu in ((3.0, 0.0), (4.0, 0.3), (6.0, -0.45), (20.0, 0.1), (2.0, 0.7), (100.0, 0.2)):
            print(f"coefficients M={m} beta'={beta} mu~={mu}", flush=True)
            c = cd.chebdm_coeffs(handle, beta, mu, -1.0, 1.0, ORDER, m)
            f = 1 / (1 + np.exp(LD(beta) * (x - LD(mu))))
            f64 = f.astype(np.float64)
            for i in range(0, n.size, 64):
                q = (n[i:i + 64, None] * j[None, :]) % (4 * m)
                ce = cosines[q]
                got.append(c[n[i:i + 64]].astype(LD) - 2 * (ce @ f) / m)
                plain = 2.0 * one_cosine_a_term(f64, cosines, q) / m
                want.append(plain.astype(LD) - 2 * (ce @ f64.astype(LD)) / m)
    handle.close()
    rms = [float(np.sqrt(np.mean(np.concatenate(e).astype(np.float64) ** 2))) for e in (got, want)]
    print("rms", rms)
    assert rms[0] <= 1.08 * rms[1]
