"""Forms of a solve that a handle takes by its data or its entry point: packed models with stored conductances (a model
whose label 0 conducts) and in label form, and steps replayed from captured graphs (spfd_solve_many) against steps
launched one by one (spfd_solve)."""
import numpy as np
import pytest

import oracle
import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_2010_12879_amd as P  # noqa: E402

DEV = torch.device("cuda:0")
BAR = {"fp64": 1e-7, "mixed": 1e-6}


def _dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).to(DEV)


def _models(dims, seed):
    ws = [W.random_ellipsoid_phantom(nx, ny, nz, seed=seed + i, n_ell=5, semi_range=(2.5, 9.0), name=f"f{i}")
          for i, (nx, ny, nz) in enumerate(dims)]
    assert all(np.any(w.labels > 0) for w in ws)
    return ws


def _check(ms, ws, tables, prec):
    """Potentials at 1e-12 against the oracle's at 1e-12, model by model, and the same bits from a second solve."""
    psis, infos = ms.solve([_dev(w.a) for w in ws], tol=1e-12, max_iter=400)
    again, infos2 = ms.solve([_dev(w.a) for w in ws], tol=1e-12, max_iter=400)
    assert infos == infos2 and all(torch.equal(p, q) for p, q in zip(psis, again))
    for k, (w, t) in enumerate(zip(ws, tables)):
        ref, _ = oracle.solve(np.asarray(t)[w.labels], w.h, w.a, tol=1e-12)
        p = psis[k].cpu().numpy()
        err = np.linalg.norm(p - ref) / np.linalg.norm(ref)
        print(f"model {k}: iterations {infos[k]['iterations']} error {err:.2e}", flush=True)
        assert infos[k]["status"] == "OK" and err <= BAR[prec]
        assert np.abs(p - ref).max() <= BAR[prec] * np.abs(ref).max()


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("dims,solid", [([(24, 20, 28), (40, 32, 48), (17, 23, 9), (33, 29, 37)], [1]),
                                        ([(24, 20, 28), (40, 32, 48), (17, 23, 9), (33, 29, 37)], [0, 2, 3]),
                                        ([(16, 24, 63), (30, 14, 63), (9, 9, 64)], [0, 1, 2]),
                                        ([(16, 24, 63), (30, 14, 63), (9, 9, 64)], []),
                                        ([(96, 80, 120), (20, 24, 31)], [0])], ids=str)
def test_packed_models_with_stored_conductances(dims, solid, prec):
    """Some models' label 0 conducts (the whole box): the finest level is stored, not in label form. Models that end at
    the node layer below the next one's first (also in label form, where the bricks around a model's are another's, with
    conductivities of another size), few bricks (own sums, legs) and more."""
    print(f"case packed stored {dims} {solid} {prec}", flush=True)
    ws = _models(dims, 330)
    tables = [np.array(w.sigma_table, dtype=np.float64) for w in ws]
    for k in solid:
        tables[k][0] = 0.07 * (k + 1)
    tables = [t * 1e-4**k for k, t in enumerate(tables)]
    ms = P.MultiSolver([_dev(w.labels) for w in ws], tables, ws[0].h, precision=prec)
    _check(ms, ws, tables, prec)
    ms.close()


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_packed_models_change_form(prec):
    """One handle: label form, then stored conductances, then label form with other tables."""
    print(f"case packed change of form {prec}", flush=True)
    ws = _models([(24, 20, 28), (40, 32, 48), (17, 23, 9)], 340)
    air = [np.array(w.sigma_table, dtype=np.float64) for w in ws]
    solid = [t.copy() for t in air]
    solid[2][0] = 0.2
    other = [t * np.linspace(0.5, 2.0, len(t)) for t in air]
    ms = P.MultiSolver([_dev(w.labels) for w in ws], air, ws[0].h, precision=prec)
    for tables in (air, solid, other):
        P.spfd_set_sigma_tables(ms.handle, [list(t) for t in tables])
        P.spfd_build(ms.handle, P.AmgOptions(P.MIXED if prec == "mixed" else P.FP64))
        _check(ms, ws, tables, prec)
    ms.close()


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("size", [(28, 24, 36), (64, 48, 56), (131, 97, 101)], ids=str)
def test_replayed_steps_equal_launched_ones(size, prec):
    """Two handles together (replayed graphs) and each alone (direct launches), with both betas in turn, so that the
    graphs are captured anew at each change, replayed over other eager work, and launched (eager): the same bits."""
    print(f"case replay {size} {prec}", flush=True)
    ws = [W.random_ellipsoid_phantom(*size, seed=61 + i, n_ell=8, semi_range=(4.0, 11.0)) for i in range(2)]
    srcs = [_dev(w.a) for w in ws]
    torch.cuda.synchronize()
    ss = [P.Solver(_dev(w.labels), w.sigma_table, w.h, precision=prec) for w in ws]
    alone = {f: [s.solve(a, tol=1e-10, flexible=f) for s, a in zip(ss, srcs)] for f in (False, True)}
    psis = [torch.empty_like(p) for p, _ in alone[False]]
    for flexible, eager in ((False, 0), (False, 0), (True, 0), (True, 0), (False, 0), (True, 1), (False, 1), (False, 0)):
        for p in psis:
            p.fill_(7.0)
        float(torch.randn(4096, device=DEV, dtype=torch.float64).sum())
        torch.cuda.synchronize()
        opts = P.SolveOptions(1e-10, 500, 0, eager, P.CG, 30, 1 if flexible else 0)
        st, infos = P.spfd_solve_many([s.handle for s in ss], opts, psis, 2)
        assert st == 0
        for k, (p, info) in enumerate(alone[flexible]):
            assert infos[k] == info, (flexible, eager, k, infos[k], info)
            assert torch.equal(psis[k], p), (flexible, eager, k)
    for s in ss:
        s.close()
