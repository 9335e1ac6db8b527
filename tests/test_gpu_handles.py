"""A handle starts from clean host scalars: its pinned memory may have been an earlier handle's, with stamps of the
same numbers, which the host must not take for this handle's kernels'."""
import numpy as np
import pytest

import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_2010_12879_amd as P  # noqa: E402

DEV = torch.device("cuda:0")


@pytest.mark.parametrize("prec", ["mixed", "fp64"])
def test_handles_one_after_another(prec):
    """The same solves on fresh handles that follow handles stopped at other steps and grown to more right sides (which
    gives the first pinned memory back early): the same bits, iterations and residual."""
    print(f"case handles {prec}", flush=True)
    w = W.random_ellipsoid_phantom(31, 29, 37, seed=11, n_ell=6, semi_range=(4.0, 9.0))
    lab, a = (torch.from_numpy(np.ascontiguousarray(v)).to(DEV) for v in (w.labels, w.a))
    want = {}
    for k in range(48):
        limit = (1, 2, 3, 4, 6, 300)[k * 5 % 6 if k % 12 < 6 else k % 6]
        s = P.Solver(lab, w.sigma_table, w.h, precision=prec)
        psi, info = s.solve(a, tol=1e-9, max_iter=limit, check=False)
        ref = want.setdefault(limit, (psi, info["iterations"], info["rel_residual"]))
        s.solve(torch.stack([a, -a, 2.0 * a]), tol=1e-9, max_iter=limit, check=False)
        s.close()
        assert (info["iterations"], info["rel_residual"]) == ref[1:], (k, limit, info, ref[1:])
        assert torch.equal(psi, ref[0]), (k, limit)
