"""Field, edge voltages and edge potentials on grids whose layers or number of layers exceed what fits a 32-bit product or one launch
dimension."""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_2010_12879_amd as P  # noqa: E402

DEV = torch.device("cuda:0")


def _free_for(nbytes):
    torch.cuda.empty_cache()
    free = torch.cuda.mem_get_info(DEV)[0]
    if free < nbytes + (8 << 30):
        pytest.skip(f"needs {nbytes / 1e9:.0f} GB of device memory, {free / 1e9:.0f} are free")


@pytest.mark.parametrize("voxel", [False, True])
@pytest.mark.parametrize("nz", [262139, 262141, 300001])
def test_many_layers(nz, voxel):
    """65,535 blocks of four layers fill a launch's y dimension; below, just above, and with a remainder.  The bound
    on u is that of its two additions, on |E| that of four edges' voltages, their sum and the square root."""
    print(f"case layers {nz} {voxel}", flush=True)
    rng = np.random.default_rng(nz)
    shape, h, omega = (nz, 2, 2), (1e-3, 2e-3, 3e-3), 3.0
    lab = rng.integers(0, 3, shape).astype(np.uint8)
    table = np.array([0.0, 0.2, 0.9])
    nodes = (nz + 1, 3, 3)
    a, psi = rng.standard_normal((3,) + nodes), rng.standard_normal(nodes)
    ud, ed = torch.full((3,) + nodes, 7.0, dtype=torch.float64, device=DEV), torch.full(shape, 7.0, dtype=torch.float64,
                                                                                       device=DEV)
    hd = P.spfd_create()
    try:
        P.spfd_set_geometry(hd, 2, 2, nz, *h, torch.from_numpy(lab).to(DEV))
        if voxel:
            P.spfd_set_sigma_voxel(hd, torch.from_numpy(table[lab]).to(DEV))
        else:
            P.spfd_set_sigma_table(hd, table)
        P.spfd_efield(hd, omega, torch.from_numpy(a).to(DEV), torch.from_numpy(psi).to(DEV), ud, ed)
    finally:
        P.spfd_destroy(hd)
    u_ref, e_ref = oracle.efield(table[lab], h, a, psi, omega)
    top = np.abs(a).max() + 2.0 * np.abs(psi).max()
    eps = np.finfo(np.float64).eps
    assert np.abs(ud.cpu().numpy() - u_ref).max() <= 4 * eps * top
    assert np.abs(ed.cpu().numpy() - e_ref).max() <= 32 * eps * omega * top / min(h)


def test_layer_of_2e31_voxels():
    """|E| of a slab one voxel thick with 46,341 x 46,341 voxels: a constant a_x and no gradient give omega a_x / hx in
    every voxel exactly (125 GB; the potentials are the plane a_x, which is constant too)."""
    n = 46341
    nodes = 2 * (n + 1) * (n + 1)
    _free_for(8 * (3 * nodes + n * n) + 2 * n * n)
    print("case layer of 2^31 voxels", flush=True)
    a = torch.zeros((3, nodes), dtype=torch.float64, device=DEV)
    a[0] = 1.0
    emag = torch.full((n * n,), -1.0, dtype=torch.float64, device=DEV)
    hd = P.spfd_create()
    try:
        P.spfd_set_geometry(hd, n, n, 1, 0.5, 1.0, 1.0, torch.ones((1, n, n), dtype=torch.uint8, device=DEV))
        P.spfd_set_sigma_table(hd, [0.0, 0.4])
        P.spfd_efield(hd, 3.0, a, a[0], None, emag)
        lo, hi = float(emag.min()), float(emag.max())
    finally:
        P.spfd_destroy(hd)
        del a, emag
        torch.cuda.empty_cache()
    assert lo == hi == 6.0, (lo, hi)


def test_edge_potentials_of_a_layer_of_2e31_columns():
    """The tree-cotree potentials of one flux b_y, at the last edge of a slab of 46,341 x 46,341 node columns: a_x above
    it is that flux, everything else 0 (207 GB)."""
    n = 46340
    nodes = 2 * (n + 1) * (n + 1)
    _free_for(8 * 6 * nodes + 2 * n * n)
    print("case edge potentials of 2^31 columns", flush=True)
    flux = torch.zeros((3, 2, n + 1, n + 1), dtype=torch.float64, device=DEV)
    a = torch.full((3, 2, n + 1, n + 1), 5.0, dtype=torch.float64, device=DEV)
    flux[1, 0, n, n - 1] = 2.0
    hd = P.spfd_create()
    try:
        P.spfd_set_geometry(hd, n, n, 1, 1.0, 1.0, 1.0, torch.zeros((1, n, n), dtype=torch.uint8, device=DEV))
        P.spfd_edge_potentials(hd, flux, a)
        got = float(a[0, 1, n, n - 1])
        a[0, 1, n, n - 1] = 0.0
        lo, hi = float(a.min()), float(a.max())
    finally:
        P.spfd_destroy(hd)
        del a, flux
        torch.cuda.empty_cache()
    assert got == 2.0 and lo == hi == 0.0, (got, lo, hi)
