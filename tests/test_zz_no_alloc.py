"""conststn_execute_static (partial row blocks in the library's static device array, nothing allocated by
the call) against conststn_execute, on two calls in a row, the second with a smaller input."""
import gc

import pytest
import torch

import paper_2401_04836_amd as cst
import workloads as w
from paper_2401_04836_amd import schedules as S

pytestmark = pytest.mark.gpu


def _plan(wl):
    dev = "cuda"
    X = wl.sparse["X"]
    csf = cst.build_csf([c.to(dev) for c in X.coords], X.vals.to(dev), X.dims, [0, 1, 2])
    U2, U3 = wl.dense["U2"].to(dev), wl.dense["U3"].to(dev)
    pl = cst.plan(S.TTMC3, [("X", csf), ("U3", U3), ("U2", U2)], flags=cst.OUT_COMPACT)
    return pl, [U3, U2]


def test_execute_static_matches_execute_twice_in_a_row():
    # a power-law tensor whose heaviest slices are cut into several work items (partial row blocks in use),
    # then a smaller one that leaves most of the array's previous contents in place
    cases = [w.make(5, small=True),
             w.make(5, small=True, dims=(3001, 2999, 509), nnz=40_009, ranks=(32, 64))]
    for n, wl in enumerate(cases):
        print("[case] execute_static call %d: %s" % (n, {k: (v.dims, v.nnz) for k, v in wl.sparse.items()}), flush=True)
        pl, facs = _plan(wl)
        assert "family=ttmc3" in pl.describe()
        assert int(pl.describe().split("partial_blocks=")[1].split()[0]) > 0     # the scratch array is in use
        want = cst.execute(pl, facs)
        got = torch.full_like(want, float("nan"))
        free_before = torch.cuda.mem_get_info()[0]
        cst.execute_static(pl, facs, got)
        torch.cuda.synchronize()
        assert torch.cuda.mem_get_info()[0] == free_before          # nothing was allocated by the call
        assert torch.equal(got, want)                               # same kernels, same order of additions
        # and once more on the same plan: the array's contents from the first run do not leak into the result
        got2 = torch.full_like(want, float("nan"))
        cst.execute_static(pl, facs, got2)
        torch.cuda.synchronize()
        assert torch.equal(got2, want)


def test_execute_static_rejects_what_it_cannot_take():
    wl = w.make(2, small=True)
    X = wl.sparse["X"]
    csf = cst.build_csf([c.cuda() for c in X.coords], X.vals.cuda(), X.dims, [0, 1, 2])
    B, C = wl.dense["B"].cuda(), wl.dense["C"].cuda()
    pl = cst.plan(S.MTTKRP3, [("X", csf), ("C", C), ("B", B)])
    out = torch.empty(pl.n_rows * pl.row_elems, dtype=torch.float64, device="cuda")
    with pytest.raises(cst.ConststnError) as e:
        cst.execute_static(pl, [C, B], out)
    assert e.value.status_name == "EUNSUPPORTED"


@pytest.mark.parametrize("ranks", [(63, 63), (50, 50), (64, 33)])
def test_execute_static_takes_a_flat_tensor_at_any_ranks(ranks):
    """300 slices of 3 300 leaves each, most of them in fibers of their own: no slice is long enough that its partial
    row blocks must exceed the array."""
    g = torch.Generator(device="cuda").manual_seed(11)
    dims, nnz = (300, 20_000, 500), 1_000_000
    keys = torch.unique(torch.randint(0, dims[0] * dims[1] * dims[2], (nnz,), generator=g, device="cuda"))
    keys = keys[torch.randperm(keys.numel(), generator=g, device="cuda")]
    coords = [x.to(torch.int32) for x in (keys // (dims[1] * dims[2]), keys // dims[2] % dims[1], keys % dims[2])]
    vals = torch.rand(keys.numel(), generator=g, dtype=torch.float64, device="cuda")
    U2, U3 = (torch.rand(d, r, generator=g, dtype=torch.float64, device="cuda") for d, r in zip(dims[1:], ranks))
    print("[case] execute_static, flat tensor, ranks %s" % (ranks,), flush=True)
    csf = cst.build_csf(coords, vals, dims, [0, 1, 2])
    pl = cst.plan(S.TTMC3, [("X", csf), ("U3", U3), ("U2", U2)])
    want = cst.execute(pl, [U3, U2])
    got = torch.full_like(want, float("nan"))
    cst.execute_static(pl, [U3, U2], got)
    torch.cuda.synchronize()
    assert torch.equal(got, want)
    general = cst.plan(S.TTMC3, [("X", csf), ("U3", U3), ("U2", U2)], options=dict(ttmc3_mfma=0))
    # positive terms, at most 3 500 per sum
    assert (cst.execute(general, [U3, U2]) / got - 1).abs().max().item() <= 4e-13


def test_memory_of_destroyed_objects_is_given_back_on_demand():
    n = 4_000_000
    coords = [torch.randperm(n, device="cuda").to(torch.int32) for _ in range(3)]
    vals = torch.rand(n, dtype=torch.float64, device="cuda")
    print("[case] build, destroy, release", flush=True)
    alive = cst.build_csf(coords, vals, (n, n, n), [0, 1, 2])
    torch.cuda.synchronize()
    gc.collect()             # handles of other tests, in the cycle of a caught exception: collected in between they give memory back too
    cst.release_memory()
    before = torch.cuda.mem_get_info()[0]
    cst.build_csf(coords, vals, (n, n, n), [1, 2, 0]).destroy()
    assert torch.cuda.mem_get_info()[0] < before              # kept for the next build
    cst.release_memory()
    assert torch.cuda.mem_get_info()[0] == before
    alive.check()
