"""The whole-side passes of 1D applies: sizes with one to five transfer levels, ragged widths, both precisions and
directions, and their splits."""
import pytest

import fio_inputs as fi
from gpu_common import fiohss, dev, host, perr, gpu_bf, oracle_bf, step

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [256, 1024, 4096])
@pytest.mark.parametrize("k", [1, 9, 40])
def test_side_passes_match_oracle(n, k):
    F = fiohss()
    step("side passes n=%d k=%d" % (n, k))
    B = gpu_bf(F, n, 9, "sin16", imported=False, precs=(F.FIO_PREC_FP64, F.FIO_PREC_FP32))
    ob = oracle_bf(n, 9, "sin16")
    x = fi.complex_gaussian(14, fi.PURPOSE_PROBE, n, k)
    # FP64: the bound of the other applies; FP32: 2^-24 per table entry, coefficient and product over
    # 2 x 5 factors of at most 18 terms, 10 x (2 + sqrt(18)) x 2^-24 < 1e-5
    for prec, tol in ((F.FIO_PREC_FP64, 1e-12), (F.FIO_PREC_FP32, 1e-5)):
        assert perr(host(B.apply(dev(x), prec=prec)), ob.apply(x)) < tol
        assert perr(host(B.apply_adj(dev(x), prec=prec)), ob.apply_adj(x)) < tol


def test_splits_and_widths_are_bitwise_equal():
    # N = 2^16 has five transfer levels a side: 70 columns write the output in the last pass, narrow blocks and
    # leaf_sep in a kernel of its own, kmax splits the side
    F = fiohss()
    import torch
    n, k = 1 << 16, 70
    step("side passes n=%d" % n)
    B = gpu_bf(F, n, 9, "sin16", imported=False, precs=(F.FIO_PREC_FP64, F.FIO_PREC_FP32))
    X = dev(fi.complex_gaussian(15, fi.PURPOSE_PROBE, n, k))
    for prec in (F.FIO_PREC_FP64, F.FIO_PREC_FP32):
        for f, adj in ((B.apply, False), (B.apply_adj, True)):
            whole = f(X, prec=prec)
            for lo, hi in ((0, 1), (1, 9), (9, 46)):
                assert torch.equal(f(X[:, lo:hi], prec=prec), whole[:, lo:hi]), (prec, adj, lo, hi)
            for kmax, sep in ((0, 1), (1, 0), (2, 1), (3, 0)):
                B.set_tile(k, prec=prec, adj=adj, kmax=kmax, leaf_sep=sep)
                assert torch.equal(f(X, prec=prec), whole), (prec, adj, kmax, sep)
            B.set_tile(k, prec=prec, adj=adj)
