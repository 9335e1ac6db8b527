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


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("shape,fill,split_level", [((20, 21, 37), 0.28, 1), ((24, 24, 24), 0.4, 1),
                                                    ((31, 40, 33), 0.22, 2), ((40, 40, 40), 0.34, 1)], ids=str)
def test_split_levels(shape, fill, split_level, prec):
    """Split levels of random sparse bodies, where pieces have many neighbours and aggregates more than eight
    members, down to a coarsest level of at most 48 unknowns: the Galerkin operators are exact, so the solve reaches
    1e-12 and agrees with the oracle's (also at 1e-12) to the condition number times that, below 1e-7."""
    print(f"case split {shape} {fill} {split_level} {prec}", flush=True)
    rng = np.random.default_rng(shape[0] + shape[2])
    lab = (rng.random(shape) < fill).astype(np.uint8) * rng.integers(1, 4, shape).astype(np.uint8)
    lab[0, 0, 0] = 1
    table, h = [0.0, 0.1, 0.6, 1.7], (2e-3, 2e-3, 3e-3)
    a = rng.standard_normal((3,) + tuple(n + 1 for n in shape))
    s = P.Solver(torch.from_numpy(lab).to(DEV), table, h, precision=prec, split_level=split_level, coarsest_max=48)
    psi, info = s.solve(torch.from_numpy(a).to(DEV), tol=1e-12, max_iter=400)
    widths = [P.spfd_level_info(s.handle, k)["row_entries"] for k in range(s.info()["n_levels"])]
    s.close()
    ref, _ = oracle.solve(np.asarray(table)[lab], h, a, tol=1e-12)
    print("row entries", widths, "iterations", info["iterations"], flush=True)
    assert info["status"] == "OK" and min(widths) == 7 and max(widths) >= 9
    assert np.linalg.norm(psi.cpu().numpy() - ref) <= 1e-7 * np.linalg.norm(ref)


@pytest.mark.parametrize("shape", [(7, 9, 16), (3, 11, 31), (4, 16, 16), (5, 5, 41), (20, 13, 4), (8, 8, 64),
                                   (241, 17, 1), (16, 17, 241)], ids=str)
def test_voxel_flags_at_wave_remainders(shape):
    """A wave reads 1,024 conductivities: voxel counts one run of 16 or one voxel below and above that, and just it, on
    a body with a conductor in its first and last voxels.  A value that is not finite or below 0 is refused wherever it
    is."""
    n = int(np.prod(shape))
    print(f"case voxel flags {shape} {n} = {n // 1024} x 1024 + {n % 1024}", flush=True)
    rng = np.random.default_rng(n)
    sig = np.where(rng.random(shape) < 0.2, rng.uniform(0.1, 1.0, shape), 0.0)
    sig.flat[0] = sig.flat[-1] = 0.3
    h = (2e-3, 2e-3, 2e-3)
    lab = torch.ones(shape, dtype=torch.uint8, device=DEV)
    s = P.Solver(lab, torch.from_numpy(sig).to(DEV), h)
    info = s.info()
    s.close()
    touched = np.zeros(tuple(m + 1 for m in shape), bool)
    for k in (0, 1):
        for j in (0, 1):
            for i in (0, 1):
                touched[k:shape[0] + k, j:shape[1] + j, i:shape[2] + i] |= sig > 0
    assert info["n_dofs"] == touched.sum()
    assert info["n_components"] == oracle.components(sig, h)[1]
    for at in (0, n // 2, n - 1):
        for bad in (-0.1, np.inf, np.nan):
            wrong = sig.copy()
            wrong.flat[at] = bad
            with pytest.raises(P.SPFDError):
                P.Solver(lab, torch.from_numpy(wrong).to(DEV), h)
