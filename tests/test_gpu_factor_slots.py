"""Setup on patterns that choose between the slot layout's direct
factorisation and the general one, and on subdomains at the edges of the level
kernels: levels bit for bit, factors to the bound of the parity tests (1e-12),
the apply of a general variant (CSR streams built on demand) and of the slot
kernel alike, and a refactorisation equal bit for bit to a fresh setup."""

import dataclasses

import numpy as np
import pytest

import oracle as O
from parity import check_close, dd_scale
from problems import Problem, laplacian_scalar, random_blocks

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover - collected on CPU machines, skipped by marker
    pytest.skip("no GPU", allow_module_level=True)

import paper_2508_04917_amd as P  # noqa: E402
from paper_2508_04917_amd.solver import DDSolver  # noqa: E402


def keep(p, mask):
    rows = np.repeat(np.arange(p.n), np.diff(p.brow_ptr))
    ptr = np.zeros(p.n + 1, dtype=np.int32)
    np.cumsum(np.bincount(rows[mask], minlength=p.n), out=ptr[1:])
    return dataclasses.replace(p, brow_ptr=ptr, bcol=p.bcol[mask], val=p.val[mask])


def one_sided(nx, ny, nz, seed):
    """A structurally unsymmetric pattern: a third of the couplings missing."""
    p = random_blocks(nx, ny, nz, seed=seed)
    rows = np.repeat(np.arange(p.n), np.diff(p.brow_ptr))
    drop = np.random.default_rng(seed).random(rows.size) < 0.33
    return keep(p, ~drop | (rows == p.bcol))


def comb(ny, seed):
    """2 x ny rows, coupled along x everywhere and along y at x = 1: ny rows
    in the first level, which the rows of the one-row levels after it reach
    back to (ny positions), so that 2 ny inverses have to stay at hand."""
    p = random_blocks(2, ny, 1, seed=seed)
    rows = np.repeat(np.arange(p.n), np.diff(p.brow_ptr))
    return keep(p, (rows // 2 == p.bcol // 2) | ((rows % 2 == 1) & (p.bcol % 2 == 1)))


def triangles(nx, ny, bs, seed):
    """Triangular mesh: three lower neighbours that couple to each other, so
    ILU0 updates off-diagonal blocks too."""
    rng = np.random.default_rng(seed)
    i, j = np.meshgrid(np.arange(nx), np.arange(ny), indexing="xy")
    g = (i + nx * j).ravel()
    rows, cols = [g], [g]
    for di, dj in ((1, 0), (0, 1), (-1, 1)):
        ok = ((i + di >= 0) & (i + di < nx) & (j + dj < ny)).ravel()
        a, b = g[ok], g[ok] + di + nx * dj
        rows += [a, b]
        cols += [b, a]
    r, c = np.concatenate(rows), np.concatenate(cols)
    o = np.lexsort((c, r))
    r, c = r[o], c[o]
    val = 0.05 * rng.standard_normal((r.size, bs, bs)) - np.eye(bs)
    val[r == c] = 7.0 * np.eye(bs) + 0.05 * rng.standard_normal((g.size, bs, bs))
    ptr = np.zeros(g.size + 1, dtype=np.int32)
    np.cumsum(np.bincount(r, minlength=g.size), out=ptr[1:])
    return Problem("triangles", nx, ny, 1, bs, ptr, c.astype(np.int32), val, rng.standard_normal(g.size * bs), seed)


CASES = {
    # name: (problem, box, factored into the slot streams directly)
    "stencil": (lambda: random_blocks(22, 18, 10, seed=41), (11, 9, 5)),
    "stencil_scalar": (lambda: laplacian_scalar(30, 20, 10, seed=42), (15, 20, 5)),
    "one_sided": (lambda: one_sided(16, 12, 10, seed=43), (8, 6, 10)),
    "triangles": (lambda: triangles(24, 20, 3, seed=44), (12, 20, 1)),
    "triangles_scalar": (lambda: triangles(64, 30, 1, seed=45), (64, 15, 1)),
    "levels_1100": (lambda: laplacian_scalar(1100, 2, 1, seed=46), (1100, 1, 1)),
    "inverses_1024": (lambda: comb(512, seed=51), (2, 512, 1)),
    "inverses_1026": (lambda: comb(513, seed=52), (2, 513, 1)),
    "inverses_2048": (lambda: comb(1024, seed=53), (2, 1024, 1)),
    "inverses_2050": (lambda: comb(1025, seed=54), (2, 1025, 1)),  # more than the LDS holds
    "rows_5000": (lambda: laplacian_scalar(25, 20, 20, seed=47), (25, 20, 10)),
    "rows_10240": (lambda: laplacian_scalar(32, 32, 20, seed=48), (32, 32, 10)),
}


@pytest.mark.parametrize("name", list(CASES))
def test_setup(name):
    make, sub = CASES[name]
    p = make()
    print(f"[factor] {name}", flush=True)
    s = DDSolver.from_problem(p, sub=sub)
    st = O.setup(p, sub)
    for which in (0, 1):
        for a, b in zip(P.dd_get_levels(s.h, which), st.levels(which)):
            assert np.array_equal(a.cpu().numpy(), b)
    ptr, col, f = P.dd_get_factors(s.h)
    assert np.array_equal(ptr.cpu().numpy(), st.tptr) and np.array_equal(col.cpu().numpy(), st.tcol)
    check_close(f.cpu().numpy(), st.f, st.bs * st.bs, 1e-12, what=name + " factors")
    r = np.random.default_rng(9).standard_normal(st.n * st.bs)
    rd = torch.as_tensor(r, device="cuda")
    z0 = s.apply(rd)
    check_close(z0.cpu().numpy(), st.apply(r), st.bs, 1e-12, what=name, scale=dd_scale(st, r))
    # the other layout of the factors, built when a variant asks for it (and its FP32 copy)
    s.set_precision(P.ddilu.DD_MIXED)
    zm = s.apply(rd)
    P.ddilu.dd_set_apply_variant(s.h, 1)
    assert torch.equal(s.apply(rd), zm)
    s.set_precision(P.ddilu.DD_FP64)
    assert torch.equal(s.apply(rd), z0)
    # new values on the pattern, both layouts kept, against a fresh handle
    q = dataclasses.replace(p, val=p.val * np.random.default_rng(8).uniform(0.9, 1.1, p.val.shape[0])[:, None, None])
    P.ddilu.ilu0_refactor(s.h, torch.as_tensor(q.val.reshape(-1), device="cuda"))
    fresh = DDSolver.from_problem(q, sub=sub)
    z1 = fresh.apply(rd)
    assert torch.equal(s.apply(rd), z1)
    P.ddilu.dd_set_apply_variant(s.h, 0)
    assert torch.equal(s.apply(rd), z1)
    assert torch.equal(P.dd_get_factors(s.h)[2], P.dd_get_factors(fresh.h)[2])
    assert torch.equal(P.ddilu.dd_spmv(s.h, rd), P.ddilu.dd_spmv(fresh.h, rd))
    s.close()
    fresh.close()
