"""The apply + product launch with more boxes than compute units, several to
one: the same solution bit for bit from run to run, and the two-launch solve's
first residuals (the sums are only grouped otherwise: 1e-12)."""

import numpy as np
import pytest

from problems import laplacian_blocks, laplacian_scalar, random_blocks

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover - collected on CPU machines, skipped by marker
    pytest.skip("no GPU", allow_module_level=True)

from paper_2508_04917_amd import ddilu as dd  # noqa: E402
from paper_2508_04917_amd.solver import DDSolver  # noqa: E402

CASES = {
    "448_boxes": (lambda: laplacian_blocks(84, 48, 80), (6, 12, 10)),
    "1188_boxes": (lambda: random_blocks(36, 88, 108, seed=3), (3, 8, 12)),
    "936_boxes": (lambda: random_blocks(45, 117, 72, seed=4), (5, 9, 9)),
    "1728_scalar_boxes": (lambda: laplacian_scalar(96, 96, 96), (8, 8, 8)),
}


@pytest.mark.parametrize("name", list(CASES))
def test_fused_solve(name):
    make, sub = CASES[name]
    p = make()
    s = DDSolver.from_problem(p, sub=sub)
    b = torch.as_tensor(np.ascontiguousarray(p.b), device="cuda").reshape(-1)
    hist = torch.empty(13, dtype=torch.float64, device="cuda")

    def solve():
        hist.fill_(float("nan"))
        x, info = None, None
        try:
            x, info = dd.bicgstab_solve(s.h, b, torch.zeros_like(b), rtol=1e-30, maxit=12)
        except dd.DDError as e:  # not converged after twelve iterations
            assert e.code == dd.DD_ENOCONV
        return x, info, hist.clone()

    dd.dd_set_residual_history(s.h, hist)
    _, _, two = solve()
    dd.dd_set_fusion(s.h, True)
    x, info, one = solve()
    assert info is None or info["fused"] == 1
    assert float((one[:4] / two[:4] - 1).abs().max()) <= 1e-12
    for _ in range(4):
        x2, _, again = solve()
        assert torch.equal(again, one)
        if x is not None:
            assert torch.equal(x, x2)
    dd.dd_set_residual_history(s.h, None)
    s.close()
