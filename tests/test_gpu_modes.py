"""Every output mode of the order-3 MTTKRP and TTMc (Sec. 5.2-5.3 run one contraction per mode)
by re-rooting the CSF: output mode at the root, the two other modes in either order below it."""
import itertools

import numpy as np
import pytest
import torch

import oracle
import workloads as w
from helpers import TOL, compare, to_dev
import paper_2401_04836_amd as cst
from paper_2401_04836_amd import schedules as S

pytestmark = pytest.mark.gpu

LEVELS = [p for p in itertools.permutations(range(3))]


def _say(msg):
    print(msg, flush=True)


def _factors(seed, dims, ranks):
    g = torch.Generator().manual_seed(seed)
    return [torch.rand(dims[m], ranks[m], generator=g, dtype=torch.float64) * 2 - 1 for m in range(3)]


@pytest.mark.parametrize("levels", LEVELS)
def test_mttkrp_every_mode_and_level_order(levels):
    wl = w.make(2, small=True)
    X = wl.sparse["X"]
    F = _factors(77, X.dims, (32, 32, 32))
    _say("mttkrp output mode %d, CSF level order %s" % (levels[0], (levels,)))
    dc, dv = to_dev(X)
    csf = cst.build_csf(dc, dv, X.dims, list(levels))
    text, names = S.mttkrp3_for(levels)
    leaf, mid = F[levels[2]].cuda(), F[levels[1]].cuda()
    pl = cst.plan(text, [(names[0], csf), (names[1], leaf), (names[2], mid)])
    out = cst.execute(pl, [leaf, mid]).reshape(pl.n_rows, -1)
    torch.cuda.synchronize()
    c, v = X.numpy()
    other = sorted(levels[1:])
    Fa, Fb = F[other[0]].numpy(), F[other[1]].numpy()
    want = oracle.mttkrp3(c, v, X.dims, Fa, Fb, levels[0])
    S_abs = oracle.mttkrp3_abs(c, v, X.dims, Fa, Fb, levels[0])
    assert compare(out, want, S_abs) <= TOL


@pytest.mark.parametrize("levels", LEVELS)
@pytest.mark.parametrize("ranks", [(8, 5, 11), (16, 32, 48)])
def test_ttmc3_every_mode_and_level_order(levels, ranks):
    wl = w.make(1)
    X = wl.sparse["X"]
    F = _factors(78, X.dims, ranks)
    _say("ttmc output mode %d, CSF level order %s, ranks %s" % (levels[0], (levels,), (ranks,)))
    dc, dv = to_dev(X)
    csf = cst.build_csf(dc, dv, X.dims, list(levels))
    text, names = S.ttmc3_for(levels)
    leaf, mid = F[levels[2]].cuda(), F[levels[1]].cuda()
    pl = cst.plan(text, [(names[0], csf), (names[1], leaf), (names[2], mid)])
    out = cst.execute(pl, [leaf, mid]).reshape(pl.n_rows, mid.shape[1], leaf.shape[1])
    torch.cuda.synchronize()
    c, v = X.numpy()
    other = sorted(levels[1:])
    Fa, Fb = F[other[0]].numpy(), F[other[1]].numpy()
    want = oracle.ttmc3(c, v, X.dims, Fa, Fb, levels[0])            # [root, R_other0, R_other1]
    S_abs = oracle.ttmc3_abs(c, v, X.dims, Fa, Fb, levels[0])
    if levels[1] > levels[2]:                                       # GPU rows are [middle, leaf]
        out = out.permute(0, 2, 1).contiguous()
    assert compare(out, want, S_abs) <= TOL


# the three trees whose result is indexed by a level below the root, X stored i > j > k
NOT_THE_ROOT = [("T[i,j,r] = X[i,j,k] * C[k,r] | i,j,k,r ; M[j,r] = T[i,j,r] * A[i,r] | i,j,r", 1, ("C", "A")),
                ("T[i,j,k,r] = X[i,j,k] * A[i,r] | i,j,k,r ; M[k,r] = T[i,j,k,r] * B[j,r] | i,j,k,r", 2, ("A", "B")),
                ("T[i,j,k,r] = X[i,j,k] * B[j,r] | i,j,k,r ; M[k,r] = T[i,j,k,r] * A[i,r] | i,j,k,r", 2, ("B", "A"))]


@pytest.mark.parametrize("rank", [1, 2, 128])
@pytest.mark.parametrize("text,mode,names", NOT_THE_ROOT)
def test_mttkrp_of_a_level_below_the_root_at_the_smallest_ranks(text, mode, names, rank):
    """The result is [extent of its mode, rank] and the same in every run; compact rows are those of its own mode."""
    wl = w.make(2, small=True, dims=(301, 211, 503), nnz=20_003, rank=rank)
    X = wl.sparse["X"]
    F = dict(zip("ABC", _factors(79, X.dims, (rank,) * 3)))
    _say("mttkrp of level %d, rank %d" % (mode, rank))
    dc, dv = to_dev(X)
    csf = cst.build_csf(dc, dv, X.dims, [0, 1, 2])
    dev = [F[n].cuda() for n in names]
    c, v = X.numpy()
    Fa, Fb = (F["ABC"[m]].numpy() for m in range(3) if m != mode)
    want = oracle.mttkrp3(c, v, X.dims, Fa, Fb, mode)
    S_abs = oracle.mttkrp3_abs(c, v, X.dims, Fa, Fb, mode)
    for flags in (0, cst.OUT_COMPACT):
        pl = cst.plan(text, [("X", csf)] + list(zip(names, dev)), flags=flags)
        rows = pl.output_rows() if flags else None
        assert (pl.n_rows, pl.row_elems) == (len(np.unique(c[mode])) if flags else X.dims[mode], rank)
        pl.check()
        out = cst.execute(pl, dev).reshape(pl.n_rows, rank)
        assert compare(out, want, S_abs, rows=rows) <= TOL
        for _ in range(5):
            assert torch.equal(cst.execute(pl, dev).reshape(pl.n_rows, rank), out)


def test_mttkrp_over_a_mode_of_more_than_2_28_indices():
    """A middle mode beyond what a 28-bit index names, as the root's neighbour and below the result's level."""
    dims, n, R = ((1 << 28) + 77, 40, 50), 30_011, 2
    g = torch.Generator(device="cuda").manual_seed(5)
    c = [torch.randint(0, d, (n,), generator=g, device="cuda", dtype=torch.int32) for d in dims]
    c[0][:4] = torch.tensor([0, dims[0] - 1, (1 << 28) - 1, 1 << 28], dtype=torch.int32)
    v = torch.rand(n, generator=g, dtype=torch.float64, device="cuda") + 0.5
    A = torch.rand(dims[0], R, generator=g, dtype=torch.float64, device="cuda")
    B, C = (torch.rand(d, R, generator=g, dtype=torch.float64, device="cuda") for d in dims[1:])
    _say("mttkrp over a mode of %d indices" % dims[0])
    a, b, ck = (f[x.long()] for f, x in zip((A, B, C), c))
    csf = cst.build_csf(c, v, dims, [1, 0, 2], flags=cst.COALESCE_DUPS)                    # j > i > k
    for text, names, terms, at, rows in (
            ("T[j,i,r] = X[j,i,k] * C[k,r] | j,i,k,r ; M[j,r] = T[j,i,r] * A[i,r] | j,i,r", ("C", "A"), v[:, None] * ck * a, c[1], 40),
            ("T[j,i,k,r] = X[j,i,k] * A[i,r] | j,i,k,r ; M[k,r] = T[j,i,k,r] * B[j,r] | j,i,k,r", ("A", "B"), v[:, None] * a * b, c[2], 50)):
        dev = [dict(A=A, B=B, C=C)[m] for m in names]
        pl = cst.plan(text, [("X", csf)] + list(zip(names, dev)))
        assert (pl.n_rows, pl.row_elems) == (rows, R)
        pl.check()
        got = cst.execute(pl, dev).reshape(rows, R)
        want = torch.zeros(rows, R, dtype=torch.float64, device="cuda").index_add_(0, at.long(), terms)
        assert (got / want - 1).abs().max().item() <= 1e-12        # sums of about 700 positive terms


@pytest.mark.parametrize("flags", [0, cst.OUT_COMPACT])
def test_rank_one_over_more_than_2_24_slices(flags):
    """As many slices as a launch of one workgroup each does not take: two leaves per slice, a heavy slice among them."""
    n, dims = (1 << 24) + 5000, ((1 << 24) + 70_000, 40, 30)
    g = torch.Generator(device="cuda").manual_seed(6)
    i = torch.cat([torch.randperm(dims[0], generator=g, device="cuda")[:n], torch.full((60_000,), 12_345, device="cuda")])
    j, k = (torch.randint(0, d, (i.numel(),), generator=g, device="cuda") for d in dims[1:])
    v = torch.rand(i.numel(), generator=g, dtype=torch.float64, device="cuda") + 0.5
    B, C = (torch.rand(d, 1, generator=g, dtype=torch.float64, device="cuda") for d in dims[1:])
    _say("mttkrp of rank 1 over %d slices" % n)
    csf = cst.build_csf([x.to(torch.int32) for x in (i, j, k)], v, dims, [0, 1, 2], flags=cst.COALESCE_DUPS)
    pl = cst.plan(S.MTTKRP3, [("X", csf), ("C", C), ("B", B)], flags=flags)
    pl.check()
    got = cst.execute(pl, [C, B])
    want = torch.zeros(dims[0], dtype=torch.float64, device="cuda").index_add_(0, i, v * B[j, 0] * C[k, 0])
    if flags:
        want = want[pl.output_rows().long()]
    scale = want.abs().clamp(min=1e-300)
    assert ((got - want).abs() / scale).max().item() <= 1.4e-11      # positive terms, at most 60 001 of them
