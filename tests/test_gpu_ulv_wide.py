"""The level products of the ULV solve for wide blocks and for levels of many nodes: nodes around the edges of the row
tiles, blocks around those of the column groups."""
import numpy as np
import pytest

import fio_inputs as fi
from oracle import hss as ohss, ulv as oulv
from gpu_common import fiohss, dev, host, hss_generators, perr, step

pytestmark = pytest.mark.gpu


def generators(leaf, depth, r):
    """A well conditioned HPD matrix: diagonal blocks around 8 I, orthonormal bases, small couplings."""
    h = ohss.HSS(leaf << depth, leaf)
    for l in range(1, depth + 1):
        h.rank[l] = [r] * (1 << l)
    for l in range(1, depth + 1):
        m = leaf if l == depth else 2 * r
        h.U[l] = [np.linalg.qr(fi.complex_gaussian(j, fi.PURPOSE_DATA, m, r, level=l))[0] for j in range(1 << l)]
    for l in range(depth):
        h.B[l] = [fi.complex_gaussian(j, fi.PURPOSE_DATA, r, r, level=100 + l) / (4 * r) for j in range(1 << l)]
    h.D = []
    for j in range(1 << depth):
        a = fi.complex_gaussian(j, fi.PURPOSE_DATA, leaf, leaf, level=200) / np.sqrt(leaf)
        h.D.append(8 * np.eye(leaf) + a + a.conj().T)
    return h


# 128 leaves of up to 16, 32, 64 and more rows (the last two row groups of 64); 16 and 32 leaves of more than 64 rows,
# whose inner dimension is split into slices
@pytest.mark.parametrize("leaf,depth,r,k", [(9, 7, 3, 130), (16, 7, 4, 130), (17, 7, 4, 130), (32, 7, 4, 130),
                                            (33, 7, 4, 130), (64, 7, 8, 130), (65, 7, 8, 130), (100, 7, 8, 130),
                                            (130, 5, 8, 200), (200, 4, 8, 260)])
def test_wide_blocks(leaf, depth, r, k):
    F = fiohss()
    import torch
    step("ULV solve leaf=%d depth=%d k=%d" % (leaf, depth, k))
    ho = generators(leaf, depth, r)
    n = leaf << depth
    H = F.HSS.from_generators(n, leaf, *hss_generators(ho))
    U = F.ULV(H)
    x = fi.complex_gaussian(6, fi.PURPOSE_PROBE, n, k)
    X = dev(x)
    whole = U.solve(X)
    # a column is summed in one order at every width: 1, 8, 16, 33, 48 and 65 columns
    for lo, hi in ((0, 1), (1, 9), (9, 25), (25, 58), (58, 106), (65, 130)):
        assert torch.equal(U.solve(X[:, lo:hi]), whole[:, lo:hi]), (lo, hi)
    # in place, and a leading dimension beyond n
    buf = F.empty(n + 3, k)
    buf[:n] = X
    U.solve(buf[:n], out=buf[:n])
    assert torch.equal(buf[:n], whole)
    # the bound of the other solves against the oracle
    c = [0, k // 2, k - 1]
    assert perr(host(whole)[:, c], oulv.solve(oulv.factor(ho), x[:, c])) < 1e-12
    # H c = x: a few hundred roundings of a matrix of condition under 10
    assert perr(host(H.matvec(whole)), x) < 1e-12
