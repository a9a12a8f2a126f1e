"""Inputs that are not numbers reach the result: no reflector drops a column that holds a NaN, whether a level runs one
workgroup per node or level-wide blocks."""
import numpy as np
import pytest

import fio_inputs as fi
from oracle import hss as ohss
from gpu_common import fiohss, dev, hss_generators, omega_np, step

pytestmark = pytest.mark.gpu


# 2 x 40 rows + p samples: panels of 8 columns; p = 2050 and 5300: panels of 4 and of one column
@pytest.mark.parametrize("p", [5, 2050, 5300])
def test_nan_in_the_test_matrix(p):
    from test_oracle_hss import block_structured_hermitian
    F = fiohss()
    import torch
    step("HSS construction with a NaN in Omega, p=%d" % p)
    leaf, n = 40, 160
    Hd = dev(block_structured_hermitian(n, leaf, 4, seed=31))

    def omega(l, r, c):
        om = omega_np(32)(l, r, c)
        if l == 2:
            om[45, 3] = np.nan                             # node 1 of the leaf level
        return om
    F.set_hss_big_node(1)
    try:
        H = F.HSS.from_samples(n, lambda X: Hd @ torch.nan_to_num(X), tol=1e-10, p=p, leaf=leaf, norm_est=1.0,
                               omega=F.omega_from(omega))
    finally:
        F.set_hss_big_node(0)
    # the samples of the other nodes are numbers: they have the operator's rank, node 1 has no basis
    assert [int(r) for r in H.ranks()[2]] == [8, 0, 8, 8]


@pytest.mark.parametrize("rows", [1, 4096])
@pytest.mark.parametrize("row,col", [(0, 7), (39, 7), (9, 0)])
def test_nan_in_a_basis_is_not_factored(rows, row, col):
    from test_oracle_hss import block_structured_hermitian
    F = fiohss()
    step("ULV of a basis with a NaN at (%d, %d), rows=%d" % (row, col, rows))
    leaf, n = 40, 160
    Hm = block_structured_hermitian(n, leaf, 4, seed=33)
    ho = ohss.build(n, lambda X: Hm @ X, omega_np(34), tol=1e-13, p=5, leaf=leaf)
    ho.U[2][1] = ho.U[2][1].copy()
    ho.U[2][1][row, col] = np.nan
    ranks, gen = hss_generators(ho)
    H = F.HSS.from_generators(n, leaf, ranks, gen)
    F.set_ulv_big_node(rows)
    try:
        with pytest.raises(F.FioError) as e:
            F.ULV(H)
    finally:
        F.set_ulv_big_node(0)
    assert e.value.status == -4                            # not positive definite
