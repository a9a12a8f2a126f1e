"""2D FP32 applies of q = 10 and 11, whose blocks of 16 columns keep all row tiles in one wave."""
import pytest

import fio_inputs as fi
from gpu_common import fiohss, dev, host, perr, step

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("q", [10, 11])
def test_all_row_tiles_in_a_wave(q):
    F = fiohss()
    import torch
    n, k = 32, 70
    step("2D FP32 row tiles q=%d" % q)
    B = F.BF(n, q, 2.0 / 16, 1.0 / 16, precs=(F.FIO_PREC_FP64, F.FIO_PREC_FP32), dim=2)
    X = dev(fi.complex_gaussian(7, fi.PURPOSE_PROBE, n * n, k))
    for f, adj in ((B.apply, False), (B.apply_adj, True)):
        whole = f(X, prec=F.FIO_PREC_FP32)
        # three steps of at most 16 x 121 terms, 2^-24 each: 3 x (2 + sqrt(1936)) x 2^-24 < 1e-5
        assert perr(host(whole), host(f(X))) < 1e-5
        for lo, hi in ((0, 1), (1, 17), (17, 41), (41, 70)):
            assert torch.equal(f(X[:, lo:hi], prec=F.FIO_PREC_FP32), whole[:, lo:hi]), (adj, lo, hi)
        for kc in (8, 16):
            B.set_tile(k, prec=F.FIO_PREC_FP32, adj=adj, kc=kc)
            assert torch.equal(f(X, prec=F.FIO_PREC_FP32), whole), (adj, kc)
        B.set_tile(k, prec=F.FIO_PREC_FP32, adj=adj)
