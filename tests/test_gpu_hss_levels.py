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


# the solve's kernels: levels of at most 8 rows in bands (the leaves too for leaf = 8 and 5; N = 2^12 .. 2^16 have a
# band of 1, 3 and 3 + 2 levels below the top one), up to 64 rows a wave per tile, beyond that split sums
@pytest.mark.parametrize("kind,leaf,r,depth", [("dense", 5, 1, 1), ("dense", 8, 1, 3), ("dense", 33, 4, 2),
                                               ("dense", 65, 20, 2), ("dense", 97, 40, 1),
                                               ("fio", 64, 0, 12), ("fio", 64, 0, 14), ("fio", 32, 0, 16)])
def test_solve_kernels(kind, leaf, r, depth):
    import torch
    from oracle import ulv as oulv
    from gpu_common import hss_generators
    from test_oracle_hss import block_structured_hermitian
    F = fiohss()
    step("ULV solve kernels %s leaf=%d depth=%d" % (kind, leaf, depth))
    if kind == "dense":
        n = leaf << depth
        Hm = block_structured_hermitian(n, leaf, r, seed=13)
        ho = ohss.build(n, lambda X: Hm @ X, omega_np(23), tol=1e-13, p=5, leaf=leaf)
        H = F.HSS.from_generators(n, leaf, *hss_generators(ho))
    else:
        n = 1 << depth
        H = F.HSS.from_bf(F.BF(n, 9, 2.0 / 16, 1.0 / 16), tol=1e-3, p=10, leaf=leaf, seed=4)
    U = F.ULV(H)
    x = fi.complex_gaussian(5, fi.PURPOSE_PROBE, n, 70)
    X = dev(x)
    whole = U.solve(X)
    # a column is summed in one order at every width
    for lo, hi in ((0, 1), (1, 9), (9, 26), (26, 70)):
        assert torch.equal(U.solve(X[:, lo:hi]), whole[:, lo:hi]), (lo, hi)
    if kind == "dense":
        assert perr(host(whole), oulv.solve(oulv.factor(ho), x)) < 1e-12
    # H c = x: a backward stable solve of a well conditioned H leaves a few hundred roundings
    assert perr(host(H.matvec(whole)), x) < 1e-11
