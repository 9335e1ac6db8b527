"""FGMRES columns at the edges of the basis kernels' row counts (4, 8, 16, 32 rows per pass) and of the grid."""
import numpy as np
import pytest

import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_2010_12879_amd as P  # noqa: E402

DEV = torch.device("cuda:0")


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("restart", [2, 3, 4, 5, 8, 9, 16, 17, 32])
def test_cycle_lengths(restart, prec):
    """Restart lengths (one column per cycle stagnates on this system), against CG.  Both meet the true residual 1e-11; the condition number of this phantom's
    scaled operator is below 1e5, so the two differ by less than 2e-6 at most (1e-8 seen is ordinary).  A weak
    smoother makes the cycle converge slowly enough to fill the longest one."""
    print(f"case fgmres cycle {restart} {prec}", flush=True)
    w = W.random_ellipsoid_phantom(45, 38, 52, seed=47, n_ell=10, semi_range=(3.0, 10.0))
    a = torch.from_numpy(np.ascontiguousarray(w.a)).to(DEV)
    s = P.Solver(torch.from_numpy(w.labels).to(DEV), w.sigma_table, w.h, precision=prec, smoother="l1jacobi",
                 smooth_degree=1, split=False)
    ref, _ = s.solve(a, tol=1e-11, max_iter=500)
    psi, info = s.solve(a, tol=1e-11, max_iter=2000, method="fgmres", restart=restart)
    zero, none = s.solve(torch.zeros_like(a), tol=1e-11, method="fgmres", restart=restart)
    s.close()
    assert info["status"] == "OK" and info["rel_residual"] <= 1e-11, info
    if restart > 16:
        assert info["iterations"] > 16, info
    assert torch.linalg.norm(psi - ref) <= 2e-6 * torch.linalg.norm(ref)
    assert none["status"] == "OK" and none["iterations"] == 0 and not zero.any()
