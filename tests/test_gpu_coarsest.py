"""The dense coarsest level (tiles of 64, inverted one step per launch) at the edges of its tiles: boxes small enough
to be one level, so that the cycle is the dense inverse itself."""
import numpy as np
import pytest

from tests import discrete as D

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_2010_12879_amd as P  # noqa: E402

DEV = torch.device("cuda:0")


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("shape,cut", [((1, 1, 1), None), ((2, 2, 6), None), ((3, 3, 3), None), ((1, 4, 6), None),
                                       ((7, 7, 1), None), ((4, 2, 8), None), ((9, 9, 9), None), ((7, 7, 15), None),
                                       ((7, 7, 14), 6), ((15, 7, 7), 8)], ids=str)
def test_one_level_box_is_solved_directly(shape, cut, prec):
    """n = 8, 63, 64, 70, 128, 135, 1000, 1024 unknowns; two bodies of 960 and of 1024 together.
    a = -G psi* has the answer psi* up to a constant per body.  The relative error of G psi is at most the
    condition number (12 / (2 - 2 cos(pi / 16)) = 312) times the residual 1e-12; an inverse exact to a few
    hundred roundings needs one step (two for the check of the first), an FP32 one three or four."""
    print(f"case coarsest {shape} {cut} {prec}", flush=True)
    nz, ny, nx = shape
    lab = np.ones(shape, np.uint8)
    if cut is not None:
        lab[(slice(None),) * int(np.argmax(shape)) + (cut,)] = 0
    rng = np.random.default_rng(sum(shape))
    a = -D.grad(rng.standard_normal((nz + 1, ny + 1, nx + 1)))
    s = P.Solver(torch.from_numpy(lab).to(DEV), [0.0, 0.7], (2e-3, 2e-3, 2e-3), precision=prec)
    assert s.info()["n_levels"] == 1
    psi, info = s.solve(torch.from_numpy(a).to(DEV), tol=1e-12, max_iter=50)
    s.close()
    assert info["status"] == "OK" and info["iterations"] <= (2 if prec == "fp64" else 4), info
    # edges that touch a conducting voxel
    pad = np.pad(lab, 1)
    on = [sum(pad[1 - k:nz + 2 - k, 1 - j:ny + 2 - j, 1 - i:nx + 2 - i] for i, j, k in offs) > 0 for offs in
          ([(0, j, k) for j in (0, 1) for k in (0, 1)], [(i, 0, k) for i in (0, 1) for k in (0, 1)],
           [(i, j, 0) for i in (0, 1) for j in (0, 1)])]
    got, want = D.grad(psi.cpu().numpy()), -a
    for d in range(3):
        assert np.linalg.norm((got - want)[d][on[d]]) <= 1e-9 * np.linalg.norm(want[d][on[d]])
