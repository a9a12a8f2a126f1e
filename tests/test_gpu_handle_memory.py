"""Device memory kept between handles: blocks of a destroyed handle that kernels still use, several threads
and streams, and the bound on what is kept."""
import threading

import pytest

import fio_inputs as fi
from gpu_common import fiohss, dev, step

pytestmark = pytest.mark.gpu


def test_reused_blocks_wait_for_the_kernels_that_use_them():
    F = fiohss()
    import torch
    step("handles destroyed with applies in flight")
    n, k = 1 << 14, 64
    x = dev(fi.complex_gaussian(5, fi.PURPOSE_PROBE, n, k))
    ref = F.BF(n, 9, 2.0 / 16, 1.0 / 16).apply(x)
    side = torch.cuda.Stream()
    for _ in range(4):
        B = F.BF(n, 9, 2.0 / 16, 1.0 / 16)
        ws = torch.empty(B.workspace_size(k), dtype=torch.uint8, device="cuda")
        outs = [F.empty(n, k) for _ in range(6)]
        torch.cuda.synchronize()
        with torch.cuda.stream(side):
            for o in outs:
                B.apply(x, out=o, ws=ws)
        del B                                              # its factors go back while the applies run
        F.BF(n, 9, 1.0 / 16, 2.0 / 16)                     # and are overwritten by another operator's
        torch.cuda.synchronize()
        for o in outs:
            assert torch.equal(o, ref)


def test_threads_and_bound():
    F = fiohss()
    import torch
    step("handles built by three threads")
    torch.cuda.synchronize()
    sizes = [1 << 10, 1 << 12, 1 << 14]
    want, got, errors = {}, {}, []

    def one(n, results, key):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                for _ in range(3):
                    B = F.BF(n, 9, 2.0 / 16, 1.0 / 16)
                    U = F.ULV(F.HSS.from_bf(B, tol=1e-3, p=10, seed=3))
                    f, _ = F.approx_solve(B, U, dev(fi.rhs(7, n, 4)))
                    torch.cuda.current_stream().synchronize()
                results[key] = f.clone()
                torch.cuda.current_stream().synchronize()
        except Exception as e:      # reported by the main thread
            errors.append(e)

    for n in sizes:
        one(n, want, n)
    free0 = torch.cuda.mem_get_info()[0]
    ts = [threading.Thread(target=one, args=(n, got, n)) for n in sizes]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not errors
    for n in sizes:
        assert torch.equal(got[n], want[n])
    assert free0 - torch.cuda.mem_get_info()[0] < 8 << 30


def test_tables_fill_blocks_larger_than_asked_for():
    """Offset tables of more than a block (1 MiB), on device blocks kept from buffers of 1.05 to 1.2 MiB."""
    F = fiohss()
    import torch
    step("tables on kept blocks")
    Y = dev(fi.rhs(9, 1 << 16, 2))
    want = None
    for k in (0, 1, 2, 3):
        # handles with buffers a little above 1 MiB, which the tables of the next construction may take
        small = [F.HSS.from_bf(F.BF(1 << 10, 9, 2.0 / 16, 1.0 / 16), tol=1e-3, p=p, seed=5) for p in (8, 12, 16, 20)]
        del small
        B = F.BF(1 << 16, 9, 2.0 / 16, 1.0 / 16)
        U = F.ULV(F.HSS.from_bf(B, tol=1e-3, p=10, seed=6, leaf=16))
        got, _ = F.approx_solve(B, U, Y)
        want = got if want is None else want
        assert torch.equal(got, want)
