"""One launch per leg of the cycle (small levels) against one launch per smoothing step: a source solved alone
(few workgroups: legs) and in a batch large enough that every level takes the separate kernels must give the
same bits, on every kind of operator, degree, coarser level and precision the legs have."""
import numpy as np
import pytest

import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_2010_12879_amd as P  # noqa: E402

DEV = torch.device("cuda:0")
MOST = 512   # workgroups (bricks x right sides) above which no level runs legs


def _dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).to(DEV)


@pytest.mark.parametrize("prec", ["mixed", "fp64"])
@pytest.mark.parametrize("opts", [{}, {"voxel": True}, {"level1_degree": 2}, {"level1_fp32": True}, {"split": False},
                                  {"smooth_degree": 4, "coarsest_max": 48}, {"coarsest_max": 48},
                                  {"split_level": 1, "coarsest_max": 48}, {"smoother": "chebyshev4"},
                                  {"smoother": "l1jacobi", "voxel": True}], ids=str)
def test_legs_equal_separate_kernels(opts, prec):
    print(f"case legs {opts} {prec}", flush=True)
    opts = dict(opts)
    voxel = opts.pop("voxel", False)
    w = W.random_ellipsoid_phantom(45, 38, 52, seed=47, n_ell=10, semi_range=(3.0, 10.0))
    sig = _dev(w.sigma_voxel() * np.random.default_rng(3).uniform(0.8, 1.2, w.labels.shape)) if voxel else w.sigma_table
    s = P.Solver(_dev(w.labels), sig, w.h, precision=prec, **opts)
    bricks = [s_["slots"] // 512 for s_ in (P.spfd_level_info(s.handle, k) for k in range(s.info()["n_levels"]))
              if s_["kind"] == "structured"]
    assert bricks[0] <= 256, bricks               # alone, every structured level runs legs
    n = MOST // bricks[-1] + 1 if len(bricks) == 1 else MOST // min(bricks) + 1
    n = min(n, 80)
    assert n * bricks[min(1, len(bricks) - 1)] > MOST, (n, bricks)   # the batch: not the finest nor the first coarse one
    a = _dev(w.a)
    srcs = torch.stack([a * (1.0 + 0.01 * k) for k in range(n)])
    one, info = s.solve(srcs[1].contiguous(), tol=1e-10, max_iter=300)
    many, infos = s.solve(srcs, tol=1e-10, max_iter=300)
    s.close()
    assert info["status"] == "OK" and infos[1]["iterations"] == info["iterations"]
    assert torch.equal(one, many[1])


@pytest.mark.parametrize("prec", ["mixed", "fp64"])
@pytest.mark.parametrize("opts", [{}, {"voxel": True}, {"level1_degree": 2}, {"coarsest_max": 48}, {"level1_fp32": True},
                                  {"smoother": "chebyshev4", "split_level": 1, "coarsest_max": 48}], ids=str)
def test_eighths_equal_whole_bricks(opts, prec):
    """A source alone on few bricks (levels dealt out in eighths of bricks) and in a batch of three (whole bricks on
    the larger levels) or of 48 (on all of them): the same bits."""
    print(f"case leg eighths {opts} {prec}", flush=True)
    opts = dict(opts)
    voxel = opts.pop("voxel", False)
    w = W.random_ellipsoid_phantom(31, 29, 37, seed=11, n_ell=6, semi_range=(4.0, 9.0))
    sig = _dev(w.sigma_voxel() * np.random.default_rng(3).uniform(0.8, 1.2, w.labels.shape)) if voxel else w.sigma_table
    s = P.Solver(_dev(w.labels), sig, w.h, precision=prec, **opts)
    bricks = [s_["slots"] // 512 for s_ in (P.spfd_level_info(s.handle, k) for k in range(s.info()["n_levels"]))
              if s_["kind"] == "structured"]
    assert bricks[0] > 16 and bricks[1] <= 48, bricks
    a = _dev(w.a)
    one, info = s.solve((a * 1.01).contiguous(), tol=1e-10, max_iter=300)
    for n in (3, 48):
        many, infos = s.solve(torch.stack([a * (1.0 + 0.01 * k) for k in range(n)]), tol=1e-10, max_iter=300)
        assert infos[1]["iterations"] == info["iterations"]
        assert torch.equal(one, many[1])
    s.close()
    assert info["status"] == "OK"


@pytest.mark.parametrize("prec", ["mixed", "fp64"])
@pytest.mark.parametrize("window", [0, 2, 4])
@pytest.mark.parametrize("max_iter", [1, 2, 3, 6, 300])
def test_residual_sums_left_to_the_next_leg(max_iter, window, prec):
    """A source alone (the sum of ||r||^2 formed beside the next step's first leg) and in a batch large enough that
    the finisher forms it: the same iterations, status and bits, stopped by the limit, by the tolerance, and with x
    updated every second and fourth step."""
    print(f"case leg residual sums {max_iter} {window} {prec}", flush=True)
    w = W.random_ellipsoid_phantom(31, 29, 37, seed=11, n_ell=6, semi_range=(4.0, 9.0))
    s = P.Solver(_dev(w.labels), w.sigma_table, w.h, precision=prec, cg_window=window)
    a = _dev(w.a)
    n = 30
    assert s.info()["n_levels"] > 1 and n * P.spfd_level_info(s.handle, 0)["slots"] // 512 > MOST
    one, info = s.solve((a * 1.01).contiguous(), tol=1e-9, max_iter=max_iter, check=False)
    many, infos = s.solve(torch.stack([a * (1.0 + 0.01 * k) for k in range(n)]), tol=1e-9, max_iter=max_iter,
                          check=False)
    s.close()
    assert info["status"] == infos[1]["status"] == ("OK" if max_iter == 300 else "NOT_CONVERGED")
    assert info["iterations"] == infos[1]["iterations"] and (max_iter == 300 or info["iterations"] == max_iter)
    assert info["rel_residual"] == infos[1]["rel_residual"] and torch.equal(one, many[1])
