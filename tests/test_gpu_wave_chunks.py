"""The slot kernel's wave-chunks where they can go wrong: a wavefront with
more chunks than its table register holds (64), levels wider than a workgroup,
chunk remainders of one row, boxes of fewer chunks than wavefronts.  Against
the oracle apply, to the FP64 bound of the parity tests (1e-12; FP32 factors
with FP64 arithmetic 1e-10 against the rounded factors)."""

import dataclasses

import numpy as np
import pytest

import oracle as O
from parity import check_close, dd_scale
from problems import laplacian_scalar, random_blocks

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover - collected on CPU machines, skipped by marker
    pytest.skip("no GPU", allow_module_level=True)

import paper_2508_04917_amd as P  # noqa: E402
from paper_2508_04917_amd.solver import DDSolver  # noqa: E402


def pairs(nx, ny, nz, seed):
    """Only rows 2k and 2k+1 coupled: two levels of half the rows each."""
    p = random_blocks(nx, ny, nz, seed=seed)
    rows = np.repeat(np.arange(p.n), np.diff(p.brow_ptr))
    keep = rows // 2 == p.bcol // 2
    ptr = np.zeros(p.n + 1, dtype=np.int32)
    np.cumsum(np.bincount(rows[keep], minlength=p.n), out=ptr[1:])
    return dataclasses.replace(p, brow_ptr=ptr, bcol=p.bcol[keep], val=p.val[keep])


CASES = {
    "line_700_levels": (lambda: laplacian_scalar(700, 1, 1, seed=31), (700, 1, 1)),
    "line_blocks": (lambda: random_blocks(300, 2, 1, seed=32), (150, 1, 1)),
    "wide_levels": (lambda: pairs(40, 32, 5, seed=33), (40, 32, 5)),
    "wide_levels_many": (lambda: pairs(22, 40, 30, seed=34), (22, 10, 1)),
    "one_row_remainder": (lambda: random_blocks(22, 4, 4, seed=35), (22, 2, 1)),
    "tiny_boxes": (lambda: random_blocks(24, 24, 24, seed=36), (2, 2, 2)),
}


@pytest.mark.parametrize("name", list(CASES))
def test_apply(name):
    make, sub = CASES[name]
    p = make()
    print(f"[wave chunks] {name}", flush=True)
    s = DDSolver.from_problem(p, sub=sub)
    st = O.setup(p, sub)
    r = np.random.default_rng(7).standard_normal(st.n * st.bs)
    rd = torch.as_tensor(r, device="cuda")
    check_close(s.apply(rd).cpu().numpy(), st.apply(r), st.bs, 1e-12, what=name, scale=dd_scale(st, r))
    s.set_precision(P.ddilu.DD_MIXED)
    check_close(s.apply(rd).cpu().numpy(), st.apply_fp32_factors(r, round_input=False), st.bs, 1e-10, what=name + " mixed")
    s.close()


@pytest.mark.parametrize("bs", [3, 1])
@pytest.mark.parametrize("k", [1, 2, 3, 4, 5, 6, 7, 8, 9, 70])
def test_one_wavefront(k, bs):
    """Workgroups of one wavefront: 272 boxes of a line of k rows, one chunk a
    level, whatever remainder the prefetch depth leaves."""
    p = random_blocks(k, 17, 16, seed=37) if bs == 3 else laplacian_scalar(k, 17, 16, seed=37)
    s = DDSolver.from_problem(p, sub=(k, 1, 1))
    st = O.setup(p, (k, 1, 1))
    r = np.random.default_rng(8).standard_normal(st.n * st.bs)
    rd = torch.as_tensor(r, device="cuda")
    check_close(s.apply(rd).cpu().numpy(), st.apply(r), st.bs, 1e-12, what=f"line {k}", scale=dd_scale(st, r))
    s.set_precision(P.ddilu.DD_MIXED)
    check_close(s.apply(rd).cpu().numpy(), st.apply_fp32_factors(r, round_input=False), st.bs, 1e-10, what=f"line {k} mixed")
    s.close()


def test_sixteen_boxes_a_cu():
    """Levels of more rows than a wavefront takes, on one wavefront a box."""
    p = pairs(44, 64, 61, seed=38)
    s = DDSolver.from_problem(p, sub=(44, 1, 1))
    st = O.setup(p, (44, 1, 1))
    r = np.random.default_rng(9).standard_normal(st.n * st.bs)
    rd = torch.as_tensor(r, device="cuda")
    check_close(s.apply(rd).cpu().numpy(), st.apply(r), st.bs, 1e-12, what="pairs", scale=dd_scale(st, r))
    s.close()
