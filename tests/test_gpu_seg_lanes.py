"""Wavefronts of the segmented apply: 27-point operators whose levels and box
counts ask for 1 to 16 of them, against the plain level loop (variant 1), which
adds a row's products in another order (FP64 bound of the parity tests,
1e-12; FP32 factors are the same numbers on both sides)."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover - collected on CPU machines, skipped by marker
    pytest.skip("no GPU", allow_module_level=True)

from paper_2508_04917_amd import ddilu as dd  # noqa: E402


def cu(a, dt=torch.float64):
    return torch.as_tensor(np.ascontiguousarray(a), device="cuda").to(dt).reshape(-1)


def stencil27(nx, ny, nz, bs, seed):
    rng = np.random.default_rng(seed)
    n = nx * ny * nz
    g = np.arange(n)
    i, j, k = g % nx, g // nx % ny, g // (nx * ny)
    I, J = [], []
    for dz in (-1, 0, 1):
        for dy in (-1, 0, 1):
            for dx in (-1, 0, 1):
                ok = (i + dx >= 0) & (i + dx < nx) & (j + dy >= 0) & (j + dy < ny) & (k + dz >= 0) & (k + dz < nz)
                I.append(g[ok])
                J.append((g + dx + nx * (dy + ny * dz))[ok])
    I, J = np.concatenate(I), np.concatenate(J)
    o = np.lexsort((J, I))
    I, J = I[o], J[o]
    val = 0.05 * rng.standard_normal((len(I), bs, bs)) - 0.5 * np.eye(bs)
    val[I == J] = 27.0 * np.eye(bs)
    ptr = np.zeros(n + 1, np.int64)
    np.cumsum(np.bincount(I, minlength=n), out=ptr[1:])
    return cu(ptr, torch.int32), cu(J, torch.int32), cu(val)


@pytest.mark.parametrize("d,sub,bs", [
    ((2, 2, 2), (2, 2, 2), 3),        # one chunk a level
    ((32, 32, 32), (4, 4, 4), 3),     # several boxes a CU
    ((16, 16, 16), (8, 8, 8), 1),     # few boxes, levels of two chunks
    ((24, 24, 24), (24, 24, 24), 1),  # one box, levels of more than eight chunks
    ((15, 13, 12), (15, 13, 12), 3),  # the same with remainders
    ((60, 60, 20), (10, 10, 5), 1),   # 144 boxes
])
def test_apply(d, sub, bs):
    h = dd.dd_partition(*d, bs, *stencil27(*d, bs, seed=51), sub=sub)
    dd.ilu0_factor(h)
    assert dd.dd_get_info(h)["apply_layout"] == 2
    r = cu(np.random.default_rng(52).standard_normal(d[0] * d[1] * d[2] * bs))
    for precision in (dd.DD_FP64, dd.DD_MIXED):
        dd.dd_set_precision(h, precision)
        z = dd.dd_trsv_apply(h, r)
        dd.dd_set_apply_variant(h, 1)
        ref = dd.dd_trsv_apply(h, r)
        dd.dd_set_apply_variant(h, 0)
        assert float((z - ref).abs().max()) <= 1e-12 * float(ref.abs().max())
    h.close()
