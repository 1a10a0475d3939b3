"""Global ILU0 in the slot layout (levels of the subdomain graph, halo rows in
LDS) and on level lists where that layout does not hold it: boxes of several
sizes, a box whose halo does not fit beside it, patterns whose factorisation
updates more than pivots, a handle without decomposed factors.  Against the
oracle's global ILU0, to the FP64 bound of the parity tests."""

import numpy as np
import pytest

import oracle as O
from parity import apply_scale, check_close
from problems import laplacian_scalar, random_blocks
from test_gpu_factor_slots import one_sided, triangles

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover - collected on CPU machines, skipped by marker
    pytest.skip("no GPU", allow_module_level=True)

import paper_2508_04917_amd as P  # noqa: E402
from paper_2508_04917_amd.solver import DDSolver  # noqa: E402

CASES = {
    "boxes": (lambda: random_blocks(18, 12, 15, seed=51), (6, 4, 5)),
    "one_box": (lambda: random_blocks(9, 8, 7, seed=52), (9, 8, 7)),
    "cells": (lambda: random_blocks(6, 5, 7, seed=53), (1, 1, 1)),
    "halo_too_large": (lambda: random_blocks(32, 40, 20, seed=54), (16, 20, 20)),
    "scalar": (lambda: laplacian_scalar(24, 20, 20, seed=55), (12, 10, 5)),
    "one_sided": (lambda: one_sided(12, 12, 10, seed=56), (4, 6, 5)),
    "triangles": (lambda: triangles(24, 20, 3, seed=57), (12, 5, 1)),
}


@pytest.mark.parametrize("name", list(CASES))
def test_global_apply(name):
    make, sub = CASES[name]
    p = make()
    print(f"[global] {name}", flush=True)
    st = O.setup(p, sub)
    bs = st.bs
    f = O.ildu0(st.n, bs, st.aptr, st.acol, O.bilu0(st.n, bs, st.aptr, st.acol, st.aval))
    R = np.random.default_rng(3).standard_normal((3, st.n * bs))
    ref = [O.apply(st.n, bs, st.aptr, st.acol, f, r) for r in R]
    scale = [apply_scale(st.n, bs, st.aptr, st.acol, f, r) for r in R]
    Rd = torch.as_tensor(R, device="cuda")

    def check(h, what):
        Z = P.ddilu.dd_global_apply(h, Rd.reshape(-1), nrhs=3).reshape(3, -1).cpu().numpy()
        for q in range(3):
            check_close(Z[q], ref[q], bs, 1e-12, what=f"{name} {what} {q}", scale=scale[q])

    s = DDSolver.from_problem(p, sub=sub)
    P.ddilu.dd_global_factor(s.h)
    check(s.h, "factored")
    # new values and the old ones again on the pattern kept
    t = lambda v: torch.as_tensor(np.ascontiguousarray(v).reshape(-1), device="cuda")  # noqa: E731
    P.ddilu.ilu0_refactor(s.h, t(2.0 * p.val))
    P.ddilu.dd_global_factor(s.h)
    P.ddilu.ilu0_refactor(s.h, t(p.val))
    P.ddilu.dd_global_factor(s.h)
    check(s.h, "refactored")
    s.close()
    # without decomposed factors, then with them
    i32 = lambda a: torch.as_tensor(np.ascontiguousarray(a), device="cuda").to(torch.int32)  # noqa: E731
    h = P.ddilu.dd_partition(p.nx, p.ny, p.nz, bs, i32(p.brow_ptr), i32(p.bcol), t(p.val), sub=sub)
    P.ddilu.dd_global_factor(h)
    check(h, "partitioned only")
    P.ddilu.ilu0_factor(h)
    P.ddilu.dd_global_factor(h)
    check(h, "factored later")
    h.close()
