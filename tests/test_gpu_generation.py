"""GPU-built 1D factors at the smallest and largest interpolation orders, against the oracle."""
import numpy as np
import pytest

from gpu_common import fiohss, gpu_bf, oracle_bf, step

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [256, 1024])
@pytest.mark.parametrize("q", [2, 3, 16])
def test_built_factors_match_oracle(n, q):
    F = fiohss()
    step("1D GPU-built factors n=%d q=%d" % (n, q))
    ref = oracle_bf(n, q, "sin16").export_factors()
    got = gpu_bf(F, n, q, "sin16", imported=False).export()
    # unimodular phases times Lagrange values: 2 x 15 factors of a Lagrange product and the phase, with a
    # rounding each on either side: 64 roundings of the largest entry
    assert np.abs(got - ref).max() < 64 * 2.0 ** -53 * max(1.0, np.abs(ref).max())
