"""Buffers that a handle lets go of are given back by every call that does so:
repeated calls, failing ones too, take no more device memory from the driver
than the first, and the handle's results stay what they were."""

import gc

import numpy as np
import pytest

from problems import random_blocks

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover - collected on CPU machines, skipped by marker
    pytest.skip("no GPU", allow_module_level=True)

from paper_2508_04917_amd import ddilu as dd  # noqa: E402

MIB = 1 << 20
N = 48


def cu(a, dt=torch.float64):
    return torch.as_tensor(np.ascontiguousarray(a), device="cuda").to(dt).reshape(-1)


def partition(p, val=None):
    return dd.dd_partition(p.nx, p.ny, p.nz, p.bs, cu(p.brow_ptr, torch.int32), cu(p.bcol, torch.int32),
                           cu(p.val) if val is None else val, sub=(8, 8, 8))


def free():
    gc.collect()
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    return torch.cuda.mem_get_info()[0]


@pytest.fixture
def empty_pool():
    gc.collect()
    dd.dd_destroy(None)
    yield
    dd.dd_destroy(None)


def test_refactor_loop_with_unscaled_factors(empty_pool):
    """Variant 7's copy of U (29 MB here) is made again after each
    refactorisation, in the same memory."""
    p = random_blocks(N, N, N, seed=3)
    h, r, val = partition(p), cu(p.b), cu(p.val)
    dd.ilu0_factor(h)
    dd.dd_set_apply_variant(h, 7)
    z = [dd.dd_trsv_apply(h, r)]
    seen = []
    for _ in range(6):
        dd.ilu0_refactor(h, val)
        z.append(dd.dd_trsv_apply(h, r, z[1] if len(z) > 1 else None))
        del z[2:]
        seen.append(free())
    assert torch.equal(z[0], z[1])
    assert seen[0] - seen[-1] < 8 * MIB
    h.close()


def test_failing_factorisations(empty_pool):
    p = random_blocks(N, N, N, seed=3)
    val = cu(p.val)
    h = partition(p, torch.zeros_like(val))
    seen = []
    for _ in range(6):
        with pytest.raises(dd.DDError) as e:
            dd.ilu0_factor(h)
        assert e.value.code == dd.DD_EZEROPIVOT
        seen.append(free())
    assert seen[0] - seen[-1] < 8 * MIB
    with pytest.raises(dd.DDError) as e:  # as before any factorisation
        dd.ilu0_refactor(h, val)
    assert e.value.code == dd.DD_ESTATE
    h.close()


@pytest.mark.parametrize("precision", [dd.DD_FP64, dd.DD_MIXED])
def test_factoring_a_factored_handle(empty_pool, precision):
    """The old factors go before the new ones are allocated; the global
    ILU0, which shares the sweeps' tables, gives the same results around it,
    also around factorisations that fail in between."""
    p = random_blocks(N, N, N, seed=4)
    h, r, val = partition(p), cu(p.b), cu(p.val)
    dd.ilu0_factor(h, precision)
    dd.dd_global_factor(h)
    z, g = dd.dd_trsv_apply(h, r), dd.dd_global_apply(h, r)
    before = free()
    for _ in range(3):
        dd.ilu0_factor(h, precision)
        assert torch.equal(dd.dd_global_apply(h, r), g)
        assert torch.equal(dd.dd_trsv_apply(h, r), z)
    assert before - free() < 8 * MIB
    with pytest.raises(dd.DDError) as e:
        dd.ilu0_refactor(h, torch.zeros_like(val))
    assert e.value.code == dd.DD_EZEROPIVOT
    with pytest.raises(dd.DDError) as e:
        dd.ilu0_factor(h, precision)  # the handle holds the zero values
    assert e.value.code == dd.DD_EZEROPIVOT
    with pytest.raises(dd.DDError) as e:
        dd.ilu0_refactor(h, val)
    assert e.value.code == dd.DD_ESTATE
    h.close()
