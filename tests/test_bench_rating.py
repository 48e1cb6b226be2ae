"""bench.py rates the products against the peak of the units that run them."""
import importlib.util
import os

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def bench():
    spec = importlib.util.spec_from_file_location("bench", os.path.join(ROOT, "bench.py"))
    mod = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(mod)
    return mod


@pytest.mark.parametrize("prec,n,achieved,peak", [("fp64", 959, 1.0, 78.6), ("fp64", 960, 1.0, None),
                                                  ("fp64", 1399, 1.0, None), ("fp64", 1400, 15.0, 5000.0),
                                                  ("fp64", None, 1.0, 78.6), ("fp32", 1000, 1.0, 157.3)])
def test_rating_by_unit(bench, prec, n, achieved, peak):
    prof = dict(gemm_ms=1.0, gemm_flop=1e9, gemm_launches=2, gemm_products=4)
    r = bench.roofline_of(prof, prec, n)
    assert r["achieved"] == achieved and r["peak"] == peak
    assert r["frac"] == (round(achieved / peak, 4) if peak else None)   # both units in one call: no one peak
