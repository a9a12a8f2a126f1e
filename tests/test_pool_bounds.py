"""The bookkeeping of the device blocks kept between handles (csrc/pool.h), compiled for the host with bounds that
the steps below exceed, and the calls that report and empty it."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2609_11520_amd", "libfiohss.so")

SRC = r"""
#include <cstdio>
#include <cstdlib>
#include "pool.h"
using namespace fio;
#define CHECK(c) do { if (!(c)) { std::printf("line %d: %s\n", __LINE__, #c); std::exit(1); } } while (0)
static char mem[64];
static bool has(const PoolBlocks &b, void *p) {
    for (const auto &x : b) if (x.second.p == p) return true;
    return false;
}
int main() {
    const size_t M = 1 << 20;
    PoolBlock b;
    size_t cap = 0;
    bool wait = false;
    {   // bytes: the least recently kept blocks leave first
        BlockPool q({10 * M, 100, 100});
        PoolBlocks out;
        for (int i = 0; i < 5; ++i) q.keep(mem + i, 3 * M, 0, out);
        CHECK(q.bytes() == 9 * M && q.count() == 3 && out.size() == 2 && has(out, mem) && has(out, mem + 1));
        q.keep(mem + 9, 10 * M, 0, out);
        CHECK(q.bytes() == 10 * M && q.count() == 1 && out.size() == 5);
        q.keep(mem + 10, 11 * M, 0, out);                 // larger than the bound: nothing stays
        CHECK(q.bytes() == 0 && q.count() == 0 && out.size() == 7);
    }
    {   // count
        BlockPool q({100 * M, 4, 100});
        PoolBlocks out;
        for (int i = 0; i < 6; ++i) q.keep(mem + i, M + i, 0, out);
        CHECK(q.count() == 4 && out.size() == 2 && has(out, mem) && has(out, mem + 1));
    }
    {   // age: kept for `age` further calls, a block kept again starts anew
        BlockPool q({100 * M, 100, 3});
        PoolBlocks out;
        q.keep(mem, M, 0, out);
        for (int i = 0; i < 2; ++i) q.end_call(out);
        q.keep(mem + 1, 2 * M, 0, out);
        CHECK(out.empty());
        q.end_call(out);
        CHECK(out.empty());
        q.end_call(out);
        CHECK(out.size() == 1 && has(out, mem) && q.bytes() == 2 * M);
        for (int i = 0; i < 2; ++i) q.end_call(out);
        CHECK(out.size() == 2 && q.bytes() == 0);
    }
    {   // trimming
        BlockPool q({100 * M, 100, 100});
        PoolBlocks out;
        for (int i = 0; i < 5; ++i) q.keep(mem + i, M, 0, out);
        q.shrink(2 * M, 100, out);
        CHECK(q.bytes() == 2 * M && out.size() == 3 && !has(out, mem + 3) && !has(out, mem + 4));
        q.shrink(0, 100, out);
        CHECK(q.bytes() == 0 && q.count() == 0 && out.size() == 5);
    }
    {   // what a request takes: the smallest that fits, at most a quarter and 64 KiB too large, of its device
        BlockPool q({100 * M, 100, 100});
        PoolBlocks out;
        q.keep(mem, 4 * M, 0, out);
        q.keep(mem + 1, 5 * M, 1, out);
        q.keep(mem + 2, 5 * M, 0, out);
        CHECK(!q.take(5 * M + 1, 0, &cap, &b, &wait) && !q.take(3 * M, 0, &cap, &b, &wait));
        CHECK(q.take(4 * M - 10, 1, &cap, &b, &wait) && b.p == mem + 1 && cap == 5 * M);
        CHECK(q.take(4 * M - 10, 0, &cap, &b, &wait) && b.p == mem && cap == 4 * M && q.bytes() == 5 * M);
    }
    {   // one wait covers the blocks kept before it began, on its device
        BlockPool q({100 * M, 100, 100});
        PoolBlocks out;
        for (int i = 0; i < 4; ++i) q.keep(mem + i, M + i * M, i == 2 ? 1 : 0, out);
        CHECK(q.take(M, 0, &cap, &b, &wait) && wait);
        const long upto = q.epoch();
        q.keep(mem + 9, 16 * M, 0, out);                  // while the device is waited for
        q.waited(0, upto);
        CHECK(q.take(2 * M, 0, &cap, &b, &wait) && !wait);
        CHECK(q.take(3 * M, 1, &cap, &b, &wait) && wait);
        CHECK(q.take(16 * M, 0, &cap, &b, &wait) && wait);
        q.waited(0, upto);                                // an older wait takes nothing back
        q.keep(mem + 9, 16 * M, 0, out);
        q.waited(0, q.epoch());
        q.waited(0, upto);
        CHECK(q.take(16 * M, 0, &cap, &b, &wait) && !wait);
    }
    return 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host compiler")
def test_bounds_and_waits(tmp_path):
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(SRC)
    inc = os.path.join(ROOT, "paper_2609_11520_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I", inc, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout


@pytest.mark.skipif(not os.path.exists(LIB), reason="library not built")
def test_nothing_is_kept_before_the_first_handle():
    import paper_2609_11520_amd as F
    assert F.memory_kept() == 0
    F.trim_memory()                       # no block: no device call
    assert F.memory_kept() == 0


@pytest.mark.gpu
def test_trim_gives_the_memory_back():
    from gpu_common import fiohss, step
    F = fiohss()
    import torch
    step("memory kept after the last handle")
    F.BF(1 << 14, 9, 2.0 / 16, 1.0 / 16)                   # loads the kernels, which take memory of their own
    F.trim_memory()
    torch.cuda.synchronize()
    assert F.memory_kept() == 0
    free0 = torch.cuda.mem_get_info()[0]
    del_me = F.BF(1 << 14, 9, 2.0 / 16, 1.0 / 16)
    held = free0 - torch.cuda.mem_get_info()[0]
    del del_me
    kept = F.memory_kept()
    # the FP64 factors of N = 2^14: 2 x 72 + 81 + 8 x 162 entries a point
    assert kept >= (1 << 14) * (144 + 81 + 8 * 162) * 16 and held >= kept * 9 // 10
    F.trim_memory(1 << 20)
    assert F.memory_kept() <= 1 << 20
    F.trim_memory()
    assert F.memory_kept() == 0
    # torch and the driver may hold a little more than before: far less than what was kept
    assert free0 - torch.cuda.mem_get_info()[0] < kept // 4


@pytest.mark.gpu
def test_an_allocation_of_the_binding_takes_the_kept_memory_back():
    from gpu_common import fiohss, step
    F = fiohss()
    import torch
    step("kept memory against torch's allocator")
    F.trim_memory()
    F.BF(1 << 14, 9, 2.0 / 16, 1.0 / 16)                   # built and destroyed
    assert F.memory_kept() > 0
    real, calls = torch.empty, []

    def full(*a, **kw):                                    # torch's allocator while the library keeps blocks
        calls.append(F.memory_kept())
        if calls[-1]:
            raise torch.cuda.OutOfMemoryError("out of memory")
        return real(*a, **kw)
    torch.empty = full
    try:
        y = F.empty(64, 2)
    finally:
        torch.empty = real
    assert y.shape == (64, 2) and calls[0] > 0 and calls[1:] == [0]
