"""A solve that breaks down leaves nothing behind in the handle's vectors, whichever form of the cycle's kernels the next
solve takes."""
import numpy as np
import pytest

import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_2010_12879_amd as P  # noqa: E402

DEV = torch.device("cuda:0")


def _dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).to(DEV)


@pytest.mark.parametrize("opts", [{}, {"split_level": 3}, {"split": False}, {"level1_degree": 2}], ids=str)
def test_solves_after_a_breakdown(opts):
    """Sources and gradients of 1e60 overflow the FP32 cycle. One right side alone runs legs, 80 run the separate
    kernels: either breaks down, and the other's next results are those from before, bit for bit. The body has single
    voxels whose eight nodes make one node of the next level, which has no conductance there, in columns that hold
    nothing else."""
    print(f"case after breakdown {opts}", flush=True)
    w = W.random_ellipsoid_phantom(47, 45, 53, seed=11, n_ell=10, semi_range=(4.0, 9.0))
    lab = np.ascontiguousarray(w.labels).copy()
    alone = 0
    for k in range(4, 50, 16):
        for j in range(4, 42, 6):
            for i in range(4, 44, 6):
                if not lab[k - 3:k + 4, j - 3:j + 4, i - 3:i + 4].any():
                    lab[k, j, i] = 1
                    alone += 1
    assert alone >= 20, alone
    s = P.Solver(_dev(lab), w.sigma_table, w.h, precision="mixed", coarsest_max=48, **opts)
    a = _dev(w.a)
    n = 80
    bricks = [P.spfd_level_info(s.handle, k)["slots"] // 512 for k in (0, 1)]
    assert s.info()["n_levels"] > 2 and bricks[0] <= 512 < n * bricks[0] and n * bricks[1] > 512, bricks
    many = torch.stack([a * (1.0 + 0.01 * k) for k in range(n)])
    psi, infos = s.solve(many, tol=1e-9)
    grad = torch.rand(lab.shape, dtype=torch.float64, device=DEV, generator=torch.Generator(DEV).manual_seed(3))
    g, _, info = s.adjoint(a, psi[0], w.omega, grad, tol=1e-9)
    assert info["status"] == "OK" and all(i["status"] == "OK" for i in infos)
    assert s.adjoint(a, psi[0], w.omega, grad * 1e60, tol=1e-9)[2]["status"] == "BREAKDOWN"
    psi2, infos2 = s.solve(many, tol=1e-9)
    assert infos2 == infos and torch.equal(psi2, psi)
    assert all(i["status"] == "BREAKDOWN" for i in s.solve(many * 1e60, tol=1e-9, check=False)[1])
    g2, _, info2 = s.adjoint(a, psi[0], w.omega, grad, tol=1e-9)
    s.close()
    assert info2 == info and torch.equal(g2, g)
