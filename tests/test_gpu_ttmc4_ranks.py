"""Order-4 TTMc on the matrix-core kernel at ranks that do not fill its tiles: the smallest, both sides of every
step of its instances (32-element parts of R2 x R3, quads of R1), odd and even, fibers and nodes from one to many
pieces, against the CPU oracle.  A guard behind the result shows that the masked stores stay inside it."""
import numpy as np
import pytest
import torch

import oracle
import paper_2401_04836_amd as cst
from paper_2401_04836_amd import schedules as S

pytestmark = pytest.mark.gpu

RANKS = [(1, 1, 1), (1, 16, 16), (16, 1, 1), (4, 2, 16), (5, 3, 11), (8, 8, 8), (7, 5, 13), (9, 13, 5), (10, 12, 7), (12, 16, 8),
         (13, 9, 15), (16, 16, 15), (15, 16, 16), (16, 16, 16)]


def _tensor(dims, nnz, seed):
    rng = np.random.default_rng(seed)
    keys = rng.permutation(np.unique(rng.integers(0, np.prod(dims), nnz)))
    c = [x.astype(np.int32) for x in np.unravel_index(keys, dims)]
    return rng, c, rng.uniform(0.5, 1, len(keys))


def _plan(c, v, dims, U, **options):
    csf = cst.build_csf([torch.from_numpy(x).cuda() for x in c], torch.from_numpy(v).cuda(), dims, [0, 1, 2, 3])
    u1, u2, u3 = (torch.from_numpy(x).cuda() for x in U)
    return cst.plan(S.TTMC4, [("X", csf), ("U3", u3), ("U2", u2), ("U1", u1)], options=options), [u3, u2, u1]


@pytest.mark.parametrize("ranks", RANKS)
@pytest.mark.parametrize("dims,nnz", [((5, 7, 6, 9), 300), ((2, 3, 40, 50), 3000), ((9, 60, 5, 3), 2000)])
def test_ranks_beside_the_tile_edges(ranks, dims, nnz):
    rng, c, v = _tensor(dims, nnz, sum(ranks))
    U = [rng.uniform(-1, 1, (d, r)) for d, r in zip(dims[1:], ranks)]
    print("[case] ranks %s dims %s nnz %d" % (ranks, dims, len(v)), flush=True)
    pl, factors = _plan(c, v, dims, U, ttmc4_ksplit=3)
    want, S_abs = oracle.ttmc4(c, v, dims, *U), oracle.ttmc4_abs(c, v, dims, *U)
    n = want.size
    buf = torch.full((n + 17,), 7.0, dtype=torch.float64, device="cuda")
    cst.execute(pl, factors, out=buf[1:1 + n])
    got = buf.cpu().numpy()
    # sums of at most 3000 products of four factors in any order: 3003 roundings of 1.1e-16
    assert oracle.rel_err(got[1:1 + n].reshape(want.shape), want, S_abs) <= 3.4e-13
    assert got[0] == 7.0 and (got[1 + n:] == 7.0).all()


@pytest.mark.parametrize("factor", [0, 1, 2])
def test_a_row_that_is_not_finite_reaches_its_own_results_only(factor):
    dims, ranks = (6, 9, 8, 7), (6, 10, 7)
    rng, c, v = _tensor(dims, 250, 3)
    U = [rng.uniform(0.5, 1, (d, r)) for d, r in zip(dims[1:], ranks)]
    U[factor][4, 2] = np.inf
    out = []
    for mfma in (0, 1):                                   # the general kernel pads nothing
        pl, factors = _plan(c, v, dims, U, ttmc4_mfma=mfma)
        out.append(cst.execute(pl, factors).cpu().numpy())
    assert np.isinf(out[0]).any() and np.isfinite(out[0]).any() and not np.isnan(out[0]).any()
    np.testing.assert_array_equal(np.isinf(out[0]), np.isinf(out[1]))
    assert not np.isnan(out[1]).any()


@pytest.mark.parametrize("ranks,longer", [((16, 16, 16), True), ((10, 12, 7), False)])
def test_items_of_a_large_tensor(ranks, longer):
    """About 0.3 M K-steps in 300 slices: at ranks 16 x 16 x 16 items of 64 K-steps (16 per slice and fewer), at smaller
    row blocks of 32."""
    g = torch.Generator(device="cuda").manual_seed(31)
    dims, n = (300, 20_000, 900, 700), 1_250_000
    keys = torch.unique(torch.randint(0, int(np.prod(np.array(dims, dtype=np.int64))), (n,), generator=g, device="cuda"))
    keys = keys[torch.randperm(keys.numel(), generator=g, device="cuda")]
    c = []
    for d in reversed(dims):
        c.append((keys % d).to(torch.int32))
        keys = keys // d
    v = torch.rand(c[0].numel(), generator=g, dtype=torch.float64, device="cuda")
    print("[case] order-4 TTMc, ranks %s, %d nonzeros" % (ranks, v.numel()), flush=True)
    csf = cst.build_csf(c[::-1], v, dims, [0, 1, 2, 3])
    U = [torch.rand(d, r, generator=g, dtype=torch.float64, device="cuda") for d, r in zip(dims[1:], ranks)]
    ops = [("X", csf)] + list(zip(("U3", "U2", "U1"), U[::-1]))
    pl, general = cst.plan(S.TTMC4, ops), cst.plan(S.TTMC4, ops, options=dict(ttmc4_mfma=0))
    blocks = int(pl.describe().split("partial_blocks=")[1].split()[0])
    assert 300 * 13 <= blocks <= 300 * 17 if longer else 300 * 26 <= blocks <= 300 * 33, blocks
    a, b = cst.execute(pl, U[::-1]), cst.execute(general, U[::-1])
    assert (a / b - 1).abs().max().item() <= 9.5e-13              # positive terms, at most 4 200 per sum
