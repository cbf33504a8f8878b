"""Order-3 TTMc on the streaming matrix-core kernel at ranks that do not fill its 16 x 32 tiles: the smallest,
one above and one below every tile edge, odd and even, against the CPU oracle.  A guard behind the result shows
that the masked stores stay inside it, and a result that is not aligned to 16 bytes is written alike."""
import numpy as np
import pytest
import torch

import oracle
import paper_2401_04836_amd as cst
from paper_2401_04836_amd import schedules as S

pytestmark = pytest.mark.gpu

RANKS = [(2, 2), (8, 8), (10, 7), (7, 10), (15, 33), (17, 31), (31, 3), (33, 64), (64, 33), (47, 49), (50, 50), (63, 63),
         (48, 50), (64, 62)]


@pytest.mark.parametrize("ranks", RANKS)
@pytest.mark.parametrize("dims,nnz", [((7, 11, 13), 300), ((1, 5, 900), 2000), ((40, 3, 50), 3000)])
def test_ranks_beside_the_tile_edges(ranks, dims, nnz):
    R2, R3 = ranks
    rng = np.random.default_rng(R2 * 100 + R3)
    keys = rng.permutation(np.unique(rng.integers(0, np.prod(dims), nnz)))
    c = [x.astype(np.int32) for x in np.unravel_index(keys, dims)]
    v = rng.uniform(-1, 1, len(keys))
    U2, U3 = rng.uniform(-1, 1, (dims[1], R2)), rng.uniform(-1, 1, (dims[2], R3))
    print("[case] ranks %s dims %s nnz %d" % (ranks, dims, len(keys)), flush=True)
    csf = cst.build_csf([torch.from_numpy(x).cuda() for x in c], torch.from_numpy(v).cuda(), dims, [0, 1, 2])
    u2, u3 = torch.from_numpy(U2).cuda(), torch.from_numpy(U3).cuda()
    pl = cst.plan(S.TTMC3, [("X", csf), ("U3", u3), ("U2", u2)], options=dict(ttmc3_rowsplit=64))
    assert "kernel=stream" in pl.describe()
    assert "producers 4" in cst.plan(S.TTMC3, [("X", csf), ("U3", u3), ("U2", u2)], options=dict(ttmc3_producers=8)).describe()
    pl.check()
    want, S_abs = oracle.ttmc3(c, v, dims, U2, U3, 0), oracle.ttmc3_abs(c, v, dims, U2, U3, 0)
    n = want.size
    for shift in (0, 1):
        buf = torch.full((n + 16,), 7.0, dtype=torch.float64, device="cuda")
        cst.execute(pl, [u3, u2], out=buf[shift:shift + n])
        got = buf.cpu().numpy()
        # sums of at most 3000 products of three factors in any order: 3002 roundings of 1.1e-16
        assert oracle.rel_err(got[shift:shift + n].reshape(want.shape), want, S_abs) <= 3.4e-13
        assert (got[:shift] == 7.0).all() and (got[shift + n:] == 7.0).all()


@pytest.mark.parametrize("ranks", [(2, 2), (7, 10), (10, 7), (33, 64), (50, 50), (63, 63)])
def test_rows_that_are_not_finite(ranks):
    """Positive terms, and a few entries of the factors that are infinite: a sum with an infinite term is infinite
    (never NaN from an absent leaf or row that is multiplied by 0), every other one is what it is without them."""
    R2, R3 = ranks
    dims = (40, 30, 50)
    rng = np.random.default_rng(R2 * 100 + R3)
    keys = rng.permutation(np.unique(rng.integers(0, np.prod(dims), 6000)))
    c = [x.astype(np.int32) for x in np.unravel_index(keys, dims)]
    v = rng.uniform(0.5, 1, len(keys))
    U2, U3 = rng.uniform(0.5, 1, (dims[1], R2)), rng.uniform(0.5, 1, (dims[2], R3))
    clean = oracle.ttmc3(c, v, dims, U2, U3, 0)
    hit2, hit3 = np.zeros_like(U2), np.zeros_like(U3)
    for hit in (hit2, hit3):
        hit[rng.integers(0, hit.shape[0], 2), rng.integers(0, hit.shape[1], 2)] = 1.0
        hit[-1, -1] = 1.0
    ones = np.ones_like
    struct = lambda a, b: oracle.ttmc3(c, ones(v), dims, a, b, 0)
    infinite = struct(hit2, ones(U3)) + struct(ones(U2), hit3) > 0
    U2[hit2 > 0], U3[hit3 > 0] = np.inf, np.inf
    print("[case] ranks %s with infinite entries" % (ranks,), flush=True)
    csf = cst.build_csf([torch.from_numpy(x).cuda() for x in c], torch.from_numpy(v).cuda(), dims, [0, 1, 2])
    u2, u3 = torch.from_numpy(U2).cuda(), torch.from_numpy(U3).cuda()
    for opts in (dict(ttmc3_rowsplit=8), {}, dict(ttmc3_mfma=0)):
        pl = cst.plan(S.TTMC3, [("X", csf), ("U3", u3), ("U2", u2)], options=opts)
        got = cst.execute(pl, [u3, u2]).cpu().numpy().reshape(clean.shape)
        assert not np.isnan(got).any(), opts
        np.testing.assert_array_equal(np.isinf(got), infinite)
        np.testing.assert_allclose(got[~infinite], clean[~infinite], rtol=1e-12)


@pytest.mark.parametrize("ranks", [(63, 63), (64, 64)])
def test_a_plan_that_does_not_fit_is_made_for_the_general_kernel(ranks):
    """Items of one row over twelve million rows ask for more partial row blocks than any device holds."""
    g = torch.Generator(device="cuda").manual_seed(12)
    dims, n = (1200, 100_000, 40_000), 13_000_000
    keys = torch.unique(torch.randint(0, dims[0] * dims[1] * dims[2], (n,), generator=g, device="cuda"))
    keys = keys[torch.randperm(keys.numel(), generator=g, device="cuda")]
    c = [x.to(torch.int32) for x in (keys // (dims[1] * dims[2]), keys // dims[2] % dims[1], keys % dims[2])]
    v = torch.rand(keys.numel(), generator=g, dtype=torch.float64, device="cuda")
    u2, u3 = (torch.rand(d, r, generator=g, dtype=torch.float64, device="cuda") for d, r in zip(dims[1:], ranks))
    print("[case] ranks %s, partial row blocks beyond the device's memory" % (ranks,), flush=True)
    csf = cst.build_csf(c, v, dims, [0, 1, 2])
    ops = [("X", csf), ("U3", u3), ("U2", u2)]
    pl = cst.plan(S.TTMC3, ops, options=dict(ttmc3_rowsplit=1))
    assert "kernel=general" in pl.describe()
    usual = cst.plan(S.TTMC3, ops)
    assert "kernel=stream" in usual.describe()
    a, b = cst.execute(pl, [u3, u2]), cst.execute(usual, [u3, u2])
    assert (a / b - 1).abs().max().item() <= 2.7e-12              # positive terms, at most 12 000 per sum


@pytest.mark.parametrize("ranks,per_slice,heavy,kernel", [((3, 40), 4, 0, "general"), ((4, 40), 4, 0, "stream"), ((3, 32), 4, 0, "stream"),
                                                          ((3, 40), 30, 0, "stream"), ((3, 40), 4, 9000, "stream"),
                                                          ((2, 8), 1, 0, "general"), ((2, 8), 5, 0, "stream"), ((3, 8), 1, 0, "stream")])
def test_short_slices_with_small_row_blocks(ranks, per_slice, heavy, kernel):
    """Row blocks that leave the streaming kernel's tiles nearly empty stay with the general kernel where slices are short and
    none is long."""
    R2, R3 = ranks
    dims = (2000, 60, 400)
    rng = np.random.default_rng(R2 * 100 + R3 + per_slice)
    keys = rng.integers(0, np.prod(dims), dims[0] * per_slice)
    if heavy:
        keys = np.concatenate([keys, 777 * 24_000 + rng.integers(0, 24_000, heavy)])
    keys = rng.permutation(np.unique(keys))
    c = [x.astype(np.int32) for x in np.unravel_index(keys, dims)]
    v = rng.uniform(-1, 1, len(keys))
    U2, U3 = rng.uniform(-1, 1, (dims[1], R2)), rng.uniform(-1, 1, (dims[2], R3))
    print("[case] ranks %s, %d leaves per slice, %d in one" % (ranks, per_slice, heavy), flush=True)
    csf = cst.build_csf([torch.from_numpy(x).cuda() for x in c], torch.from_numpy(v).cuda(), dims, [0, 1, 2])
    u2, u3 = torch.from_numpy(U2).cuda(), torch.from_numpy(U3).cuda()
    want, S_abs = oracle.ttmc3(c, v, dims, U2, U3, 0), oracle.ttmc3_abs(c, v, dims, U2, U3, 0)
    for flags in (0, cst.OUT_COMPACT):
        pl = cst.plan(S.TTMC3, [("X", csf), ("U3", u3), ("U2", u2)], flags=flags)
        assert "kernel=" + kernel in pl.describe(), pl.describe()
        rows = pl.output_rows().cpu().numpy() if flags else slice(None)
        got = cst.execute(pl, [u3, u2]).cpu().numpy().reshape(-1, R2, R3)
        assert oracle.rel_err(got, want[rows], S_abs[rows]) <= 1e-12      # at most 8000 products of three factors per sum
