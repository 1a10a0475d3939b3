"""Infinities and NaN in an apply's input: the slot kernel pads short rows
with zero blocks, which must not turn an infinite value into NaN in the global ILU0
and where levels are wider than a pass.  Against sweeps without padding: row by
row on the host with the library's factors, and for the global ILU0 its
level-scheduled form (of a handle whose decomposed sweeps are not built)."""

import numpy as np
import pytest

from problems import laplacian_scalar, random_blocks

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover - collected on CPU machines, skipped by marker
    pytest.skip("no GPU", allow_module_level=True)

from paper_2508_04917_amd import ddilu as dd  # noqa: E402



def cu(a, dt=torch.float64):
    return torch.as_tensor(np.ascontiguousarray(a), device="cuda").to(dt).reshape(-1)


def grid(p, sub):
    return lambda: dd.dd_partition(p.nx, p.ny, p.nz, p.bs, cu(p.brow_ptr, torch.int32), cu(p.bcol, torch.int32),
                                   cu(p.val), sub=sub), p.n, p.bs


def ring(n, bs, part):
    """A cycle in a random numbering: few levels, each of thousands of rows."""
    rng = np.random.default_rng(9)
    number = rng.permutation(n)
    a = np.arange(n)
    I = number[np.concatenate([a, a, a])]
    J = number[np.concatenate([a, (a + 1) % n, (a - 1) % n])]
    o = np.lexsort((J, I))
    I, J = I[o], J[o]
    val = 0.1 * rng.standard_normal((3 * n, bs, bs)) - np.eye(bs)
    val[I == J] = 4.0 * np.eye(bs)
    ptr = np.arange(0, 3 * n + 1, 3)
    return lambda: dd.dd_partition_graph(n, bs, cu(ptr, torch.int32), cu(J, torch.int32), cu(val),
                                         part_rows=part), n, bs


PROBLEMS = {
    "blocks": lambda: grid(random_blocks(12, 10, 6, seed=5), (4, 5, 3)),
    "one_box": lambda: grid(random_blocks(8, 8, 8, seed=6), (8, 8, 8)),
    "scalar": lambda: grid(laplacian_scalar(16, 16, 16), (8, 8, 8)),
    # levels wider than a pass of 1,024 lanes
    "wide": lambda: ring(8192, 3, 2048),
    "wide_scalar": lambda: ring(16384, 1, 8192),
}


def same(a, b, tol):
    """Non-finite values where the other has them and equal to them, finite
    ones within tol of the largest."""
    f, inf = torch.isfinite(b), torch.isinf(b)
    wrong = int((torch.isfinite(a) != f).sum() + (torch.isinf(a) != inf).sum())
    assert wrong == 0
    assert torch.equal(a[inf], b[inf])
    if f.any():
        assert float((a[f] - b[f]).abs().max()) <= tol * float(b[f].abs().max())


def inputs(n, bs):
    """One component of one row infinite: the first and last, an edge, the
    inside; and a NaN."""
    rng = np.random.default_rng(8)
    for row in (0, n - 1, 11, n // 2 + 5):
        for v in (np.inf, -np.inf):
            r = rng.standard_normal(n * bs)
            r[row * bs + rng.integers(bs)] = v
            yield cu(r)
    r = rng.standard_normal(n * bs)
    r[n // 3 * bs] = np.nan
    yield cu(r)


def host_apply(h, rs, bs):
    """z = inv_D y - Uhat z with y = r - L y, all inputs together (the
    library's numbering throughout)."""
    ptr, col, f = (t.cpu().numpy() for t in dd.dd_get_factors(h))
    n = len(ptr) - 1
    f = f.reshape(-1, bs, bs, 1)
    y = np.stack([r.cpu().numpy().reshape(n, bs) for r in rs], 2)
    with np.errstate(all="ignore"):
        for i in range(n):
            for q in range(ptr[i], ptr[i + 1]):
                if col[q] < i:
                    for d in range(bs):
                        y[i] -= f[q, :, d] * y[col[q]][d]
        for i in reversed(range(n)):
            acc = 0.0
            for q in range(ptr[i], ptr[i + 1]):
                if col[q] == i:
                    for d in range(bs):
                        acc = acc + f[q, :, d] * y[i][d]
            for q in range(ptr[i], ptr[i + 1]):
                if col[q] > i:
                    for d in range(bs):
                        acc = acc - f[q, :, d] * y[col[q]][d]
            y[i] = acc
    return [cu(y[:, :, k]) for k in range(len(rs))]


@pytest.mark.parametrize("name", ["wide", "wide_scalar"])
def test_apply(name):
    partition, n, bs = PROBLEMS[name]()
    h = partition()
    dd.ilu0_factor(h)
    assert dd.dd_get_info(h)["apply_layout"] == 1
    rs = list(inputs(n, bs))
    refs = host_apply(h, rs, bs)
    for precision, tol in ((dd.DD_FP64, 1e-12), (dd.DD_MIXED, 1e-4), (dd.DD_FP32, 1e-4)):
        dd.dd_set_precision(h, precision)
        for r, ref in zip(rs, refs):
            same(dd.dd_trsv_apply(h, r), ref, tol)
    h.close()


@pytest.mark.parametrize("name", sorted(PROBLEMS))
def test_global_apply(name):
    partition, n, bs = PROBLEMS[name]()
    h, ref = partition(), partition()
    dd.dd_global_factor(ref)
    dd.ilu0_factor(h)
    dd.dd_global_factor(h)
    for r in inputs(n, bs):
        same(dd.dd_global_apply(h, r), dd.dd_global_apply(ref, r), 1e-12)
    h.close()
    ref.close()
