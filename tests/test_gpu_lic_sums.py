"""Batches of right-hand sides and the sums over them where their splits can
go wrong: numbers of (subdomain, right-hand side) pairs that the eight XCDs
share unevenly, more probes than one round of the loss takes, more partial
sums than one batch of its loads.  Targets bit for bit against the applies one
by one; norms and loss against numpy sums, whose order differs: at most m
roundings of 1.1e-16 each (m <= 331,776), bound 1e-10."""

import numpy as np
import pytest

from problems import lic_init_params, lognormal_problem, probe_vectors

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover - collected on CPU machines, skipped by marker
    pytest.skip("no GPU", allow_module_level=True)

from paper_2508_04917_amd import ddilu as dd  # noqa: E402
from paper_2508_04917_amd.solver import DDSolver  # noqa: E402


@pytest.mark.parametrize("grid,sub,Q", [((8, 6, 4), (4, 6, 4), 1), ((8, 6, 4), (4, 6, 4), 3),
                                        ((12, 6, 4), (4, 6, 4), 17), ((12, 12, 12), (4, 4, 4), 33),
                                        ((48, 48, 48), (16, 16, 16), 2)])
def test_batch(grid, sub, Q):
    print(f"[lic sums] {grid} in {sub}, {Q} probes", flush=True)
    p = lognormal_problem(*grid, seed=61, sigma=1.5, corr_len=3.0)
    s = DDSolver.from_problem(p, sub=sub)
    dd.lic_setup(s.h)
    dd.dd_global_factor(s.h)
    R = torch.as_tensor(probe_vectors(61, Q, p.n * 3), device="cuda")
    Zs, den = dd.lic_targets(s.h, R)
    one = torch.stack([dd.dd_global_apply(s.h, r) for r in R])
    assert torch.equal(Zs.reshape(Q, -1), one)
    z = torch.stack([s.apply(r) for r in R])
    ref = ((z - one) ** 2).sum(dim=1)
    assert np.allclose(den.cpu().numpy(), ref.cpu().numpy(), rtol=1e-10, atol=0)
    # a network whose output layer is zero leaves the plain applies: every
    # probe's share of the loss is 1 / Q
    P = torch.as_tensor(lic_init_params(3), dtype=torch.float32, device="cuda")
    loss, _ = dd.lic_loss_grad(s.h, P, R, Zs, den)
    assert abs(float(loss.item()) - 1.0) < 1e-10
    s.close()
