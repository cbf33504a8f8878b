"""MTTKRP of order 3 and 4 on the record stream: ranks on both sides of every lane layout (2, 16, 32, 64, 96 and
128 entries per group), chunks of one block up to the default, slices inside one chunk, shared by a few chunks and
by many, empty rows, against the CPU references.  Every stream goes through the table check first; a guard behind
the result shows that the masked stores stay inside it."""
import numpy as np
import pytest
import torch

import oracle
import paper_2401_04836_amd as cst
from oracle import nary
from paper_2401_04836_amd import schedules as S

pytestmark = pytest.mark.gpu

T4 = ("T1[i,j,k,r] = X[i,j,k,l] * D[l,r] | i,j,k,l,r ; T2[i,j,r] = T1[i,j,k,r] * C[k,r] | i,j,k,r ; "
      "M[i,r] = T2[i,j,r] * B[j,r] | i,j,r")
RANKS = [2, 3, 8, 15, 16, 17, 25, 31, 32, 33, 50, 64, 65, 96, 97, 128]


def _tensor(dims, nnz, heavy, seed):
    """Distinct coordinates, `heavy` of them in the middle slice."""
    rng = np.random.default_rng(seed)
    below = int(np.prod(dims[1:]))
    keys = np.concatenate([rng.integers(0, dims[0] * below, nnz), (dims[0] // 2) * below + rng.integers(0, below, heavy)])
    keys = rng.permutation(np.unique(keys))
    return [x.astype(np.int32) for x in np.unravel_index(keys, dims)], rng.uniform(-1, 1, len(keys)), rng


def _run(text, c, v, dims, factors, opts, flags=0):
    csf = cst.build_csf([torch.from_numpy(x).cuda() for x in c], torch.from_numpy(v).cuda(), dims, list(range(len(dims))))
    dev = [torch.from_numpy(f).cuda() for _, f in factors]
    pl = cst.plan(text, [("X", csf)] + [(n, d) for (n, _), d in zip(factors, dev)], flags=flags, options=opts)
    pl.check()
    n = pl.n_rows * pl.row_elems
    buf = torch.full((n + 8,), 7.0, dtype=torch.float64, device="cuda")
    cst.execute(pl, dev, out=buf[:n])
    got = buf.cpu().numpy()
    assert (got[n:] == 7.0).all()
    return got[:n].reshape(pl.n_rows, -1), pl


@pytest.mark.parametrize("rank", RANKS)
@pytest.mark.parametrize("dims,nnz,heavy,chunk", [((7, 11, 13), 300, 0, 0), ((1, 50, 900), 20_000, 0, 16),
                                                  ((400, 30, 50), 3000, 1300, 16), ((30, 20, 40_000), 20_000, 60_000, 32)])
def test_order3(rank, dims, nnz, heavy, chunk):
    c, v, rng = _tensor(dims, nnz, heavy, 100 + rank)
    print("[case] order 3 rank %d dims %s nnz %d chunk %d" % (rank, dims, len(v), chunk), flush=True)
    B, C = rng.uniform(-1, 1, (dims[1], rank)), rng.uniform(-1, 1, (dims[2], rank))
    want, S_abs = oracle.mttkrp3(c, v, dims, B, C, 0), oracle.mttkrp3_abs(c, v, dims, B, C, 0)
    for flags in (0, cst.OUT_COMPACT):
        got, pl = _run(S.MTTKRP3, c, v, dims, [("C", C), ("B", B)], dict(mttkrp_chunk=chunk), flags)
        rows = pl.output_rows().cpu().numpy() if flags else slice(None)
        assert "kernel=records" in pl.describe()
        # at most 80 000 products of three factors per sum, in any order: 80 002 roundings of 1.1e-16
        assert oracle.rel_err(got, want[rows], S_abs[rows]) <= 8.9e-12


@pytest.mark.parametrize("rank", RANKS)
@pytest.mark.parametrize("dims,nnz,heavy,chunk", [((7, 11, 5, 13), 600, 0, 0), ((1, 5, 50, 90), 9000, 0, 16),
                                                  ((40, 8, 30, 20), 3000, 4000, 16)])
def test_order4(rank, dims, nnz, heavy, chunk):
    c, v, rng = _tensor(dims, nnz, heavy, 200 + rank)
    print("[case] order 4 rank %d dims %s nnz %d chunk %d" % (rank, dims, len(v), chunk), flush=True)
    B, C, D = (rng.uniform(-1, 1, (d, rank)) for d in dims[1:])
    got, pl = _run(T4, c, v, dims, [("D", D), ("C", C), ("B", B)], dict(mttkrp_chunk=chunk))
    assert "kernels=1 inlined_producers=2" in pl.describe() and "kernel=records" in pl.describe()
    f, ext = [(B, "jr"), (C, "kr"), (D, "lr")], {"i": dims[0], "r": rank}
    want, S_abs = nary.contract(c, v, "ijkl", f, "ir", ext), nary.contract_abs(c, v, "ijkl", f, "ir", ext)
    assert oracle.rel_err(got, want, S_abs) <= 1.0e-12       # at most 9000 products of four factors per sum



@pytest.mark.parametrize("rank", [2, 7, 25, 32, 50, 128])
@pytest.mark.parametrize("order", [3, 4])
def test_factor_rows_that_are_not_finite(order, rank):
    """Positive terms, and a few infinite entries in every factor: the sums with such a term are infinite wherever the
    chunks end -- a chunk that begins with the end of a fiber or node adds nothing of it -- and the others as without."""
    dims = (40, 8, 30, 20)[:order] if order == 4 else (40, 30, 50)
    c, _, rng = _tensor(dims, 3000, 1500, 300 + rank)
    v = rng.uniform(0.5, 1, len(c[0]))
    F = [rng.uniform(0.5, 1, (d, rank)) for d in dims[1:]]
    hits = [np.zeros_like(f) for f in F]
    for h in hits:
        h[rng.integers(0, h.shape[0], 2), rng.integers(0, rank, 2)] = 1.0
    letters = "ijkl"[:order]
    ext = {"i": dims[0], "r": rank}
    con = lambda vals, fs: nary.contract(c, vals, letters, [(f, m + "r") for f, m in zip(fs, letters[1:])], "ir", ext)
    clean = con(v, F)
    ones = [np.ones_like(f) for f in F]
    infinite = sum(con(np.ones_like(v), ones[:m] + [h] + ones[m + 1:]) for m, h in enumerate(hits)) > 0
    for f, h in zip(F, hits):
        f[h > 0] = np.inf
    names = [("B", F[0]), ("C", F[1])] if order == 3 else [("B", F[0]), ("C", F[1]), ("D", F[2])]
    for chunk in (16, 32, 48, 0):
        print("[case] order %d rank %d chunk %d with infinite entries" % (order, rank, chunk), flush=True)
        got, pl = _run(S.MTTKRP3 if order == 3 else T4, c, v, dims, names[::-1], dict(mttkrp_chunk=chunk, **({"mttkrp_split": 0} if order == 3 else {})))
        assert not np.isnan(got).any()
        np.testing.assert_array_equal(np.isinf(got), infinite)
        np.testing.assert_allclose(got[~infinite], clean[~infinite], rtol=1e-12)


def test_chunks_longer_than_the_stream():
    """A chunk length far above the number of records gives one chunk of them, not one filled up to that length."""
    dims, rank = (40, 30, 50), 32
    c, v, rng = _tensor(dims, 3000, 0, 9)
    B, C = rng.uniform(-1, 1, (dims[1], rank)), rng.uniform(-1, 1, (dims[2], rank))
    print("[case] chunks of 2^24 records over %d nonzeros" % len(v), flush=True)
    csf = cst.build_csf([torch.from_numpy(x).cuda() for x in c], torch.from_numpy(v).cuda(), dims, [0, 1, 2])
    f = [torch.from_numpy(x).cuda() for x in (C, B)]
    free = torch.cuda.mem_get_info()[0]
    pl = cst.plan(S.MTTKRP3, [("X", csf), ("C", f[0]), ("B", f[1])], options=dict(mttkrp_chunk=1 << 24))
    assert free - torch.cuda.mem_get_info()[0] < 64 << 20
    pl.check()
    got = cst.execute(pl, f).cpu().numpy().reshape(dims[0], rank)
    # at most 1500 products of three factors per sum
    assert oracle.rel_err(got, oracle.mttkrp3(c, v, dims, B, C, 0), oracle.mttkrp3_abs(c, v, dims, B, C, 0)) <= 1.7e-13


@pytest.mark.parametrize("rows,rank", [((1 << 24) + 40, 3), ((1 << 28) + 40, 2)])
def test_more_empty_rows_than_a_launch_has_threads_for(rows, rank):
    """A root mode of 2^24 to 2^28 indices of which forty hold anything: every other row is cleared."""
    dims = (rows, 30, 50)
    rng = np.random.default_rng(rows)
    at = np.sort(rng.choice(rows, 40, replace=False))
    at[-1] = rows - 1
    n = 4000
    i = rng.integers(0, 40, n)
    keys = np.unique((i * 30 + rng.integers(0, 30, n)) * 50 + rng.integers(0, 50, n))
    c = [x.astype(np.int32) for x in np.unravel_index(keys, (40, 30, 50))]
    v, B, C = rng.uniform(-1, 1, len(keys)), rng.uniform(-1, 1, (30, rank)), rng.uniform(-1, 1, (50, rank))
    want, S_abs = oracle.mttkrp3(c, v, (40, 30, 50), B, C, 0), oracle.mttkrp3_abs(c, v, (40, 30, 50), B, C, 0)
    print("[case] %d rows, rank %d" % (rows, rank), flush=True)
    csf = cst.build_csf([torch.from_numpy(x).cuda() for x in (at[c[0]].astype(np.int32), c[1], c[2])], torch.from_numpy(v).cuda(), dims, [0, 1, 2])
    f = [torch.from_numpy(x).cuda() for x in (C, B)]
    pl = cst.plan(S.MTTKRP3, [("X", csf), ("C", f[0]), ("B", f[1])])
    out = torch.full((rows * rank,), 7.0, dtype=torch.float64, device="cuda")
    cst.execute(pl, f, out=out)
    got = out.view(rows, rank)[torch.from_numpy(at).cuda()].cpu().numpy()
    assert oracle.rel_err(got, want, S_abs) <= 1.3e-14        # at most 100 products of three factors per sum
    assert int(torch.count_nonzero(out)) == np.count_nonzero(want)


@pytest.mark.parametrize("rank", [2, 3, 16, 17, 50, 128])
def test_without_a_copy_of_the_tensor(rank):
    """mttkrp_records=0: order 3 walks the CSF itself, order 4 runs on the generic executor; slices inside one chunk,
    shared by a few chunks and by many."""
    dims = (40, 30, 5000)
    c, v, rng = _tensor(dims, 3000, 20_000, 500 + rank)
    B, C = rng.uniform(-1, 1, (dims[1], rank)), rng.uniform(-1, 1, (dims[2], rank))
    want, S_abs = oracle.mttkrp3(c, v, dims, B, C, 0), oracle.mttkrp3_abs(c, v, dims, B, C, 0)
    for chunk in (0, 16):
        for flags in (0, cst.OUT_COMPACT):
            print("[case] no copy, order 3 rank %d chunk %d flags %d" % (rank, chunk, flags), flush=True)
            got, pl = _run(S.MTTKRP3, c, v, dims, [("C", C), ("B", B)], dict(mttkrp_chunk=chunk, mttkrp_records=0), flags)
            assert "kernel=csf" in pl.describe()
            rows = pl.output_rows().cpu().numpy() if flags else slice(None)
            assert oracle.rel_err(got, want[rows], S_abs[rows]) <= 2.3e-12       # at most 20 500 products of three per sum
    dims4 = (12, 8, 30, 20)
    c, v, rng = _tensor(dims4, 3000, 1500, 600 + rank)
    F = [rng.uniform(-1, 1, (d, rank)) for d in dims4[1:]]
    got, pl = _run(T4, c, v, dims4, [("D", F[2]), ("C", F[1]), ("B", F[0])], dict(mttkrp_records=0))
    f, ext = [(F[0], "jr"), (F[1], "kr"), (F[2], "lr")], {"i": dims4[0], "r": rank}
    assert oracle.rel_err(got, nary.contract(c, v, "ijkl", f, "ir", ext), nary.contract_abs(c, v, "ijkl", f, "ir", ext)) <= 4e-13


def test_an_option_at_its_default_changes_nothing():
    dims, rank = (40, 30, 500), 32
    c, v, rng = _tensor(dims, 5000, 2000, 77)
    B, C = rng.uniform(-1, 1, (dims[1], rank)), rng.uniform(-1, 1, (dims[2], rank))
    print("[case] options at their defaults", flush=True)
    base, pl = _run(S.MTTKRP3, c, v, dims, [("C", C), ("B", B)], None)
    for opts in (dict(mttkrp_hot=256), dict(mttkrp_dual=44), dict(mttkrp_split=1, mttkrp_records=1, mttkrp_chunk=0)):
        got, p = _run(S.MTTKRP3, c, v, dims, [("C", C), ("B", B)], opts)
        assert p.describe() == pl.describe() and np.array_equal(got, base), opts
    dims = (12, 8, 30, 20)
    c, v, rng = _tensor(dims, 3000, 1500, 78)
    B, C, D = (rng.uniform(-1, 1, (d, rank)) for d in dims[1:])
    base, pl = _run(T4, c, v, dims, [("D", D), ("C", C), ("B", B)], None)
    for opts in (dict(generic_span=4096), dict(generic_fuse=1, force_generic=0)):
        got, p = _run(T4, c, v, dims, [("D", D), ("C", C), ("B", B)], opts)
        assert p.describe() == pl.describe() and np.array_equal(got, base), opts
