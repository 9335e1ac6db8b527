"""spfd_percentile on fields chosen to reach every branch of its two-scan selection: values outside the
histogram window, candidate sets that fill the buffer (then the radix form runs), that fit but not in LDS,
and that are all equal; more labels than full-size histograms; grids of one scan iteration and of many.
Nearest-rank values are elements of the field, so they must equal the oracle's bit for bit."""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_2010_12879_amd as P  # noqa: E402

DEV = torch.device("cuda:0")


def _field(kind, shape, rng):
    n = int(np.prod(shape))
    if kind == "wide":           # some 60 octaves: most values below the window of the histograms
        v = np.exp(rng.normal(0.0, 8.0, n))
    elif kind == "narrow":       # one bin holds everything, values differ in the low mantissa bits
        v = 1.0 + rng.random(n) * 1e-6
    elif kind == "constant":
        v = np.full(n, 0.375)
    elif kind == "ties":
        v = rng.integers(0, 5, n).astype(np.float64)   # zeros among them
    else:
        v = np.exp(rng.normal(0.0, 1.0, n))
    return v.reshape(shape)


@pytest.mark.parametrize("kind", ["plain", "wide", "narrow", "constant", "ties"])
@pytest.mark.parametrize("shape,labels,fill", [((7, 5, 9), 3, 0.6), ((40, 37, 43), 65, 1.0), ((61, 50, 67), 66, 1.0),
                                               ((61, 50, 67), 256, 0.5), ((130, 127, 131), 41, 0.7)])
def test_percentile_branches(shape, labels, fill, kind):
    print(f"case percentile {shape} {labels} labels {kind}", flush=True)
    rng = np.random.default_rng(labels + len(kind))
    lab = (rng.integers(1, labels, shape) * (rng.random(shape) < fill)).astype(np.uint8)
    table = np.concatenate([[0.0], rng.uniform(0.1, 1.0, labels - 1)])
    table[labels // 2] = 0.0     # a label that occurs and does not conduct
    e = _field(kind, shape, rng)
    s = P.spfd_create()
    try:
        P.spfd_set_geometry(s, shape[2], shape[1], shape[0], 1e-3, 1e-3, 1e-3, torch.from_numpy(lab).to(DEV))
        sig = table[lab]
        for voxel in (False, True):
            if voxel:
                P.spfd_set_sigma_voxel(s, torch.from_numpy(sig).to(DEV))
            else:
                P.spfd_set_sigma_table(s, table)
            for q in (0.99, 0.5):
                n = 256 if voxel else labels
                body, per = P.spfd_percentile(s, torch.from_numpy(e).to(DEV), q, n)
                ref, ref_per = oracle.percentile_nearest_rank(e, lab, sig, q, n_labels=n)
                assert body == ref, (q, body, ref)
                for t in range(n):
                    assert per[t] == ref_per[t] or (np.isnan(per[t]) and np.isnan(ref_per[t])), (q, t, per[t], ref_per[t])
    finally:
        P.spfd_destroy(s)


def test_percentile_without_room_for_candidates():
    """A caller's allocator that has no block of 1 MiB left, as many as the smallest candidate buffer takes: the radix
    form answers, in the 0.3 MiB it needs, and the two-scan form once there is room again."""
    print("case percentile without room", flush=True)
    torch_alloc = P.torch_allocator(DEV)
    state = {"most": 1 << 40, "refused": 0}

    def alloc(nbytes, user):
        if nbytes > state["most"]:
            state["refused"] += 1
            return None
        return torch_alloc.alloc(nbytes, user)

    callbacks = P.Allocator(P._ALLOC_FN(alloc), P._FREE_FN(lambda p, user: torch_alloc.free(p, user)), None)
    rng = np.random.default_rng(5)
    shape = (40, 37, 43)
    lab = rng.integers(0, 5, shape).astype(np.uint8)
    table = np.array([0.0, 0.2, 0.9, 0.0, 0.4])
    e = _field("plain", shape, rng)
    s = P.spfd_create(0, None, callbacks)
    try:
        P.spfd_set_geometry(s, shape[2], shape[1], shape[0], 1e-3, 1e-3, 1e-3, torch.from_numpy(lab).to(DEV))
        P.spfd_set_sigma_table(s, table)
        ref, ref_per = oracle.percentile_nearest_rank(e, lab, table[lab], 0.99, n_labels=5)
        for most in ((1 << 20) - 1, (1 << 20) - 1, 1 << 40):
            state["most"] = most
            body, per = P.spfd_percentile(s, torch.from_numpy(e).to(DEV), 0.99, 5)
            assert body == ref
            assert all(a == b or (np.isnan(a) and np.isnan(b)) for a, b in zip(per, ref_per))
        assert state["refused"] > 0
    finally:
        P.spfd_destroy(s)
