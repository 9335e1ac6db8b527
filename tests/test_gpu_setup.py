"""Build kernels of the finest level (brick flags from runs of 16 voxels, masks, components) against the oracle's
counts on random sparse bodies whose rows are shorter than, equal to and longer than a run."""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_2010_12879_amd as P  # noqa: E402

DEV = torch.device("cuda:0")


@pytest.mark.parametrize("voxel", [False, True])
@pytest.mark.parametrize("shape,fill", [((9, 8, 1), 0.6), ((8, 7, 2), 0.5), ((19, 9, 7), 0.3), ((3, 5, 15), 0.4),
                                        ((8, 8, 16), 0.25), ((17, 24, 17), 0.15), ((33, 18, 40), 0.12),
                                        ((25, 31, 70), 0.02)], ids=str)
def test_unknowns_and_components(shape, fill, voxel):
    """Counts are exact: unknowns are the nodes of conducting voxels, components those of the edge graph."""
    print(f"case setup {shape} {fill} {voxel}", flush=True)
    rng = np.random.default_rng(shape[0] * 100 + shape[2])
    lab = (rng.random(shape) < fill).astype(np.uint8)
    lab[0, 0, 0] = 1
    h = (2e-3, 2e-3, 2e-3)
    sig = lab * 0.4
    comp, ncomp = oracle.components(sig, h)
    table = torch.from_numpy(sig).to(DEV) if voxel else [0.0, 0.4]
    s = P.Solver(torch.from_numpy(lab).to(DEV), table, h)
    info = s.info()
    s.close()
    touched = np.zeros(tuple(n + 1 for n in shape), bool)
    for k in (0, 1):
        for j in (0, 1):
            for i in (0, 1):
                touched[k:shape[0] + k, j:shape[1] + j, i:shape[2] + i] |= lab > 0
    assert info["n_dofs"] == touched.sum()
    assert info["n_components"] == ncomp
    with pytest.raises(P.SPFDError):   # the last voxel's label is not in the table
        lab[-1, -1, -1] = 7
        P.Solver(torch.from_numpy(lab).to(DEV), [0.0, 0.4], h)
