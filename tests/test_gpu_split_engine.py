"""The matrix-core engine of split precision (pinned: the default on factors built by the library are the FP32
whole-side passes): which kernels run, and its accuracy at the sizes of the solves."""
import numpy as np
import pytest

import fio_inputs as fi
from gpu_common import fiohss, dev, host, gpu_bf, oracle_bf, perr, step

pytestmark = pytest.mark.gpu
SPLIT = 2
TOL = 2e-5              # hi + lo halves with FP32 accumulation: the bound of the other split applies


def pin(B, k, **cfg):
    for adj in (False, True):
        B.set_tile(k, prec=SPLIT, adj=adj, **cfg)


def launches(F, fn):
    import torch
    torch.cuda.synchronize()
    F.timing_reset()
    F.timing_enable(True)
    try:
        y = fn()
        torch.cuda.synchronize()
    finally:
        F.timing_enable(False)
    return y, {n: F.timing_query(n)[0] for n in F.timing_names()}


# 3, 4, 5 transfer levels a side: the first pass of 3 levels folds the leaf factor in and runs in FP32, the others
# on the matrix cores
@pytest.mark.parametrize("n,k,passes", [(4096, 37, 1), (1 << 14, 64, 3), (1 << 16, 5, 3)])
def test_pinned_passes(n, k, passes):
    F = fiohss()
    step("split FP16 on the matrix cores n=%d k=%d" % (n, k))
    B = gpu_bf(F, n, 9, "sin16", imported=False, precs=(F.FIO_PREC_FP64, F.FIO_PREC_FP32, SPLIT))
    ob = oracle_bf(n, 9, "sin16")
    x = fi.complex_gaussian(41, fi.PURPOSE_PROBE, n, k)
    X = dev(x)
    for f, ref in ((B.apply, ob.apply(x)), (B.apply_adj, ob.apply_adj(x))):
        f32 = host(f(X, prec=F.FIO_PREC_FP32))
        pin(B, k, kmax=3)
        y, ran = launches(F, lambda: f(X, prec=SPLIT))
        y = host(y)
        assert ran == {"bf_struct_leaf_f32": 1, "bf_split16": passes, "bf_leaf_out_f32": 1}
        assert 1e-9 < perr(y, ref) < TOL and not np.array_equal(y, f32)
        pin(B, k, kmax=3, leaf_sep=1)
        z, ran = launches(F, lambda: f(X, prec=SPLIT))
        z = host(z)
        assert ran == {"bf_leaf_in_f32": 1, "bf_split16": passes + 1, "bf_leaf_out_f32": 1}
        assert 1e-9 < perr(z, ref) < TOL and not np.array_equal(z, y)
        # the vector units, by default and pinned, are the FP32 apply
        for cfg in ({}, dict(kmax=3, valu=1)):
            pin(B, k, **cfg)
            v, ran = launches(F, lambda: f(X, prec=SPLIT))
            assert "bf_split16" not in ran and np.array_equal(host(v), f32)
        pin(B, k)


def test_full_size_on_the_matrix_cores():
    F = fiohss()
    n, k = 1 << 18, 64
    step("split FP16 on the matrix cores n=2^18")
    B = gpu_bf(F, n, 9, "sin16", imported=False, precs=(F.FIO_PREC_FP64, F.FIO_PREC_FP32, SPLIT))
    X = dev(fi.complex_gaussian(42, fi.PURPOSE_PROBE, n, k))
    pin(B, k, kmax=3)
    for f in (B.apply, B.apply_adj):
        y, ran = launches(F, lambda: f(X, prec=SPLIT))
        assert ran["bf_split16"] == 3 and ran["bf_struct_leaf_f32"] == 1
        y, ref = host(y), host(f(X))
        assert 1e-9 < perr(y, ref) < TOL
        assert not np.array_equal(y, host(f(X, prec=F.FIO_PREC_FP32)))


def test_refinement_on_the_matrix_cores():
    F = fiohss()
    n, k = 1 << 14, 16
    step("refinement with split FP16 on the matrix cores")
    B = gpu_bf(F, n, 9, "sin16", imported=False, precs=(F.FIO_PREC_FP64, SPLIT))
    U = F.ULV(F.HSS.from_bf(B, tol=1e-3, p=10, seed=1003))
    f = fi.rhs(1, n, k)
    u = B.apply(dev(f))
    pin(B, k, kmax=3)
    (fr, info), ran = launches(F, lambda: F.approx_solve(B, U, u, mode=F.FIO_SOLVE_IR, prec=SPLIT, rel_res_tol=5e-9,
                                                         max_ir=6))
    assert ran["bf_split16"] >= 6 and info.rel_res <= 5e-9
    err = np.linalg.norm(host(fr) - f, axis=0) / np.linalg.norm(f, axis=0)
    assert err.max() < 1e-8


def test_whole_sides_with_separate_leaves_are_a_candidate():
    # 2^16 has 5 levels a side, more than any pinned pass length: the choice between leaf factors in the whole-side
    # passes and on their own is one of the tuner's
    F = fiohss()
    n, k = 1 << 16, 64
    step("autotune candidates n=2^16")
    B = gpu_bf(F, n, 9, "sin16", imported=False, precs=(F.FIO_PREC_FP64, F.FIO_PREC_FP32, SPLIT))
    X = dev(fi.complex_gaussian(43, fi.PURPOSE_PROBE, n, k))
    for prec in (F.FIO_PREC_FP64, F.FIO_PREC_FP32, SPLIT):
        rep = B.autotune(X, prec=prec, reps=1)
        assert "kmax=0 leaf_sep=0 valu=0" in rep and "kmax=0 leaf_sep=1 valu=0" in rep
