"""The construction's level-wide kernels at the edges of their blocks, against the oracle construction."""
import pytest

import fio_inputs as fi
from oracle import hss as ohss
from gpu_common import fiohss, dev, host, perr, step, omega_np

pytestmark = pytest.mark.gpu


# leaf sizes around the 8-column panels and the 32-row triangular blocks; sample counts in the three ranges of
# the panel (registers to 2048 rows in blocks of 8, to 5120 in blocks of 4, one column from memory beyond)
@pytest.mark.parametrize("leaf,depth,p", [(5, 3, 2), (16, 3, 5), (33, 3, 5), (65, 2, 7), (20, 2, 2050), (12, 2, 5300)])
def test_level_wide_construction_matches_oracle(leaf, depth, p):
    from test_oracle_hss import block_structured_hermitian
    F = fiohss()
    n = leaf << depth
    step("level-wide HSS construction leaf=%d n=%d p=%d" % (leaf, n, p))
    Hm = block_structured_hermitian(n, leaf, 4, seed=11)
    Hd = dev(Hm)
    F.set_hss_big_node(1)
    try:
        H = F.HSS.from_samples(n, lambda X: Hd @ X, tol=1e-13, p=p, leaf=leaf, omega=F.omega_from(omega_np(21)))
    finally:
        F.set_hss_big_node(0)
    ho = ohss.build(n, lambda X: Hm @ X, omega_np(21), tol=1e-13, p=p, leaf=leaf)
    assert H.ranks() == {l: list(v) for l, v in ho.rank.items()}
    x = fi.complex_gaussian(3, fi.PURPOSE_PROBE, n, 2)
    # the bound of the exact-recovery test of the default construction
    assert perr(host(H.matvec(dev(x))), Hm @ x) < 1e-11


# node sizes around the 32-row blocks of the row sweep and the 8-column blocks of the elimination; the root
# has 2 ranks' rows
@pytest.mark.parametrize("leaf,r,depth", [(5, 2, 3), (31, 4, 2), (32, 8, 3), (33, 9, 2), (64, 31, 2), (97, 33, 1)])
def test_level_wide_factorization_matches_oracle(leaf, r, depth):
    from oracle import ulv as oulv
    from gpu_common import hss_generators
    from test_oracle_hss import block_structured_hermitian
    F = fiohss()
    n = leaf << depth
    step("level-wide ULV factorization leaf=%d n=%d" % (leaf, n))
    Hm = block_structured_hermitian(n, leaf, r, seed=12)
    ho = ohss.build(n, lambda X: Hm @ X, omega_np(22), tol=1e-13, p=5, leaf=leaf)
    ranks, gen = hss_generators(ho)
    F.set_ulv_big_node(1)
    try:
        U = F.ULV(F.HSS.from_generators(n, leaf, ranks, gen))
    finally:
        F.set_ulv_big_node(0)
    x = fi.complex_gaussian(5, fi.PURPOSE_PROBE, n, 3)
    # the bound of the default factorization against the oracle
    assert perr(host(U.solve(dev(x))), oulv.solve(oulv.factor(ho), x)) < 1e-12
