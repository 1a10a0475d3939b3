"""Device memory kept between handles: results of handles built from recycled
buffers, by two threads on streams of their own, equal bit for bit those of the
first; dd_destroy(NULL) returns the memory to the driver."""

import gc
import threading

import numpy as np
import pytest

from problems import random_blocks

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover - collected on CPU machines, skipped by marker
    pytest.skip("no GPU", allow_module_level=True)

import paper_2508_04917_amd as P  # noqa: E402


def one(p, r, stream):
    t = lambda a, d: torch.as_tensor(np.ascontiguousarray(a)).to("cuda", d).reshape(-1)  # noqa: E731
    with torch.cuda.stream(stream):
        h = P.ddilu.dd_partition(p.nx, p.ny, p.nz, p.bs, t(p.brow_ptr, torch.int32), t(p.bcol, torch.int32),
                                 t(p.val, torch.float64), sub=(8, 8, 8))
        P.ddilu.ilu0_factor(h)
        z = P.ddilu.dd_trsv_apply(h, r)
        x, info = P.ddilu.bicgstab_solve(h, r)
        stream.synchronize()
        h.close()
    return z.cpu(), x.cpu(), info["iters"]


def test_recycled_buffers():
    problems = [random_blocks(24, 16, 16, seed=71), random_blocks(16, 16, 32, seed=72)]
    rs = [torch.as_tensor(p.b, device="cuda") for p in problems]
    P.ddilu.lib().dd_destroy(None)
    ref = [one(p, r, torch.cuda.Stream()) for p, r in zip(problems, rs)]
    bad = []

    def work(k):
        stream = torch.cuda.Stream()
        for i in range(6):
            j = (k + i) % 2
            got = one(problems[j], rs[j], stream)
            if not (torch.equal(got[0], ref[j][0]) and torch.equal(got[1], ref[j][1]) and got[2] == ref[j][2]):
                bad.append((k, i))

    threads = [threading.Thread(target=work, args=(k,)) for k in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not bad


def test_memory_given_back():
    gc.collect()  # handles and tensors of earlier tests
    torch.cuda.empty_cache()
    P.ddilu.lib().dd_destroy(None)
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    p = random_blocks(48, 48, 48, seed=73)
    one(p, torch.as_tensor(p.b, device="cuda"), torch.cuda.Stream())
    torch.cuda.empty_cache()
    kept = before - torch.cuda.mem_get_info()[0]
    P.ddilu.lib().dd_destroy(None)
    assert kept > 100 << 20  # the handle's buffers were still held
    assert before - torch.cuda.mem_get_info()[0] < kept // 4


def test_full_pool_keeps_the_newest():
    """With the pool full of smaller buffers, a larger handle's memory stays
    for the next one of its size: the second takes nothing from the driver."""
    gc.collect()
    torch.cuda.empty_cache()
    P.ddilu.lib().dd_destroy(None)

    def build(p):
        t = lambda a, d: torch.as_tensor(np.ascontiguousarray(a)).to("cuda", d).reshape(-1)  # noqa: E731
        args = (t(p.brow_ptr, torch.int32), t(p.bcol, torch.int32), t(p.val, torch.float64))
        return lambda: P.ddilu.dd_partition(p.nx, p.ny, p.nz, p.bs, *args, sub=(8, 8, 8))

    def free():
        torch.cuda.synchronize()
        return torch.cuda.mem_get_info()[0]

    small, large = build(random_blocks(56, 56, 56, seed=73)), build(random_blocks(80, 80, 80, seed=74))
    start, bound = free(), torch.cuda.mem_get_info()[1] // 16
    handles = []
    while start - free() < bound and len(handles) < 200:
        handles.append(small())
    for h in handles:
        h.close()
    large().close()
    before = free()
    h = large()
    assert before - free() < 64 << 20
    h.close()
    P.ddilu.lib().dd_destroy(None)
