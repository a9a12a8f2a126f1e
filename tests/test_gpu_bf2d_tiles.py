"""The 2D apply kernel at the edges of its row and column tiles, its rules for rows per wave and for the
gathered input."""
import numpy as np
import pytest

import fio_inputs as fi
from oracle import bf2d as obf2, fio2d as of2
from gpu_common import fiohss, dev, host, perr, step

pytestmark = pytest.mark.gpu


# q^2 = 4 .. 121 rows (1 to 8 row tiles, inner dimensions of every remainder mod 4), ragged widths
@pytest.mark.parametrize("n,q", [(4, 2), (8, 3), (16, 6), (8, 9), (16, 11)])
@pytest.mark.parametrize("k", [1, 9, 17])
def test_tiles_match_oracle(n, q, k):
    F = fiohss()
    step("2D tiles n=%d q=%d k=%d" % (n, q, k))
    ob = obf2.BF2D(n, q, of2.PHASE2_ANISO16)
    a0, a1 = of2.PHASE2_ANISO16
    B = F.BF(n, q, a0, a1, precs=(F.FIO_PREC_FP64, F.FIO_PREC_FP32), dim=2, factors=ob.export_factors())
    x = fi.complex_gaussian(3, fi.PURPOSE_PROBE, n * n, k)
    ref = {False: ob.apply(x), True: ob.apply_adj(x)}
    # FP64: the bound of the other 2D applies; FP32: 2^-24 per factor entry, input and rounding of sums of
    # at most 16 x 121 terms in three steps, 3 x (2 + sqrt(1936)) x 2^-24 < 1e-5
    for prec, tol in ((F.FIO_PREC_FP64, 1e-12), (F.FIO_PREC_FP32, 1e-5)):
        for adj in (False, True):
            for kc, ns in ((0, 0), (8, 1), (16, 0)):
                B.set_tile(k, prec=prec, adj=adj, kc=kc, nsplit=ns)
                got = host((B.apply_adj if adj else B.apply)(dev(x), prec=prec))
                assert perr(got, ref[adj]) < tol, (prec, adj, kc, ns)


# a column is summed in the same order whatever the width, rows per wave and input route (n = 128 has the
# single column group that runs 6 row tiles per wave, n >= 64 the gathered input from 8 columns on)
@pytest.mark.parametrize("n", [8, 32, 64, 128])
def test_columns_do_not_depend_on_the_width(n):
    F = fiohss()
    import torch
    step("2D column independence n=%d" % n)
    precs = (F.FIO_PREC_FP64,) if n == 128 else (F.FIO_PREC_FP64, F.FIO_PREC_FP32)
    B = F.BF(n, 9, 2.0 / 16, 1.0 / 16, precs=precs, dim=2)
    X = dev(fi.complex_gaussian(4, fi.PURPOSE_PROBE, n * n, 25))
    for prec in precs:
        for f, adj in ((B.apply, False), (B.apply_adj, True)):
            whole = f(X, prec=prec)
            for lo, hi in ((0, 8), (8, 9), (9, 25)):
                assert torch.equal(f(X[:, lo:hi], prec=prec), whole[:, lo:hi]), (prec, adj, lo, hi)
            B.set_tile(25, prec=prec, adj=adj, kc=16)
            assert torch.equal(f(X, prec=prec), whole)
            B.set_tile(25, prec=prec, adj=adj)
