"""The whole-side passes that end in the output rows, at widths that select them, against the leaf kernels."""
import numpy as np
import pytest

import fio_inputs as fi
from gpu_common import fiohss, dev, host, perr, step, PHASES

pytestmark = pytest.mark.gpu


# 2^16 has 256 leaf box sets: 16 chunks of 8 columns reach every threshold (4096 workgroups for the FP64 forward
# apply); the last chunk is ragged, and with an amplitude the middle blocks are read per pair
@pytest.mark.parametrize("amp", [False, True])
def test_output_pass(amp):
    F = fiohss()
    import torch
    n, k = 1 << 16, 123
    step("output rows in the last side pass, amplitude %s" % amp)
    rng = np.random.default_rng(3)
    a = (rng.uniform(0, 1, 3), rng.uniform(-0.5, 0.5, 3), 0.05) if amp else None
    B = F.BF(n, 9, *PHASES["sin16"], precs=(F.FIO_PREC_FP64, F.FIO_PREC_FP32), amp=a)
    X = dev(fi.complex_gaussian(16, fi.PURPOSE_PROBE, n, k))
    for f, adj in ((B.apply, False), (B.apply_adj, True)):
        F.set_fused(False)                                 # one kernel per factor, from the explicit factors
        try:
            ref = host(f(X))
        finally:
            F.set_fused(True)
        # FP64: the bound of the other applies; FP32: as for the whole-side passes
        for prec, kind, tol in ((F.FIO_PREC_FP64, "f64", 1e-12), (F.FIO_PREC_FP32, "f32", 1e-5)):
            torch.cuda.synchronize()
            F.timing_reset()
            F.timing_enable(True)
            y = f(X, prec=prec)
            torch.cuda.synchronize()
            F.timing_enable(False)
            if amp and not adj and kind == "f32":          # two blocks of 81 entries per partner: the leaf kernel
                assert sorted(F.timing_names()) == ["bf_leaf_out_f32", "bf_side_f32", "bf_side_in_f32"]
            else:
                assert sorted(F.timing_names()) == ["bf_side_in_" + kind, "bf_side_out_" + kind]
            assert perr(host(y), ref) < tol
            B.set_tile(k, prec=prec, adj=adj, leaf_sep=1)
            assert torch.equal(f(X, prec=prec), y), (adj, prec)
            B.set_tile(k, prec=prec, adj=adj)
            # an output with a leading dimension beyond n
            buf = F.empty(n + 5, k)
            f(X, prec=prec, out=buf[:n])
            assert torch.equal(buf[:n], y), (adj, prec)
