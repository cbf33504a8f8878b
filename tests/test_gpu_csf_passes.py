"""CSF builds whose sort takes one to six passes of 8 or 9 bits, at numbers of nonzeros beside the sort's tiles (6144 pairs;
4096 before) and their rounds over the eight XCDs, without and with duplicates (added in input order), and with a coordinate
out of range in the last place, bit for bit against the reference build."""
import numpy as np
import pytest
import torch

import paper_2401_04836_amd as cst
from oracle.csf_ref import csf_build

pytestmark = pytest.mark.gpu

# extents: 1, 7, 8, 9, 10, 17, 18, 25, 43 and 48 key bits
DIMS = [(2, 1, 1), (4, 8, 4), (8, 4, 8), (8, 8, 8), (3, 100, 2), (64, 32, 64), (64, 50, 60), (300, 200, 400),
        (12_000, 9_000, 29_000), (1 << 16, 3, (1 << 30) - 1)]


@pytest.mark.parametrize("dims", DIMS)
@pytest.mark.parametrize("n", [2, 4095, 4096, 4097, 8 * 4096, 8 * 4096 + 1, 70_001])
def test_passes_and_tiles(dims, n):
    rng = np.random.default_rng(n + sum(dims))
    c = [rng.integers(0, d, n).astype(np.int32) for d in dims]
    v = rng.uniform(-1, 1, n)
    order = [1, 2, 0]
    print("[case] dims %s n %d" % (dims, n), flush=True)
    lev = [c[m].astype(np.int64) for m in order]
    at = np.lexsort(lev[::-1])                             # stable: equal tuples keep input order
    head = np.ones(n, bool)
    head[1:] = np.any([x[at][1:] != x[at][:-1] for x in lev], axis=0)
    first = np.flatnonzero(head)
    sums = v[at][first].copy()
    for d in range(1, int(np.diff(np.append(first, n)).max())):      # one more duplicate of every tuple at a time
        more = (first + d < n) & (d < np.diff(np.append(first, n)))
        sums[more] += v[at][first[more] + d]
    idx, ptr, vals, _ = csf_build([x[at][first].astype(np.int32) for x in c], sums, dims, order)
    csf = cst.build_csf([torch.from_numpy(x).cuda() for x in c], torch.from_numpy(v).cuda(), dims, order, flags=cst.COALESCE_DUPS)
    for l in range(3):
        gi, gp, gv = csf.export(l)
        np.testing.assert_array_equal(gi.cpu().numpy(), idx[l])
        if l < 2:
            np.testing.assert_array_equal(gp.cpu().numpy(), ptr[l])
        else:
            np.testing.assert_array_equal(gv.cpu().numpy(), vals)
    c[2][n - 1] = dims[2]
    with pytest.raises(Exception, match="below its mode extent"):
        cst.build_csf([torch.from_numpy(x).cuda() for x in c], torch.from_numpy(v).cuda(), dims, order, flags=cst.COALESCE_DUPS)


@pytest.mark.parametrize("dims", [DIMS[0], DIMS[3], DIMS[7], DIMS[8], DIMS[9]])
@pytest.mark.parametrize("n", [767, 769, 6143, 6144, 6145, 8 * 6144, 8 * 6144 + 1, 9 * 6144 - 1])
def test_wavefronts_and_tiles_of_6144(dims, n):
    """Beside a wavefront's share (768 pairs) and a tile of the sort; 2 x 1 x 1: every pair of a tile in one or two digits."""
    test_passes_and_tiles(dims, n)


@pytest.mark.parametrize("bad", [-1, 1, 7, 2 ** 31 - 1])
@pytest.mark.parametrize("at", [0, 4999])
def test_range_of_a_level_without_key_bits(bad, at):
    """Fields that fill exactly 64 key bits below an outer mode of extent 1, which then holds no bit of the key: its
    coordinates are tested all the same."""
    dims, n = (1, 1 << 22, 1 << 21, 1 << 21), 5000
    rng = np.random.default_rng(7)
    c = [rng.integers(0, d, n).astype(np.int32) for d in dims]
    v = rng.uniform(-1, 1, n)
    print("[case] 64 key bits, %d at %d of mode 0" % (bad, at), flush=True)
    order = np.lexsort([x.astype(np.int64) for x in c[::-1]])
    csf = cst.build_csf([torch.from_numpy(x).cuda() for x in c], torch.from_numpy(v).cuda(), dims, [0, 1, 2, 3])
    csf.check()
    np.testing.assert_array_equal(csf.export(3)[2].cpu().numpy(), v[order])
    c[0][at] = bad
    with pytest.raises(cst.ConststnError) as e:
        cst.build_csf([torch.from_numpy(x).cuda() for x in c], torch.from_numpy(v).cuda(), dims, [0, 1, 2, 3])
    assert e.value.status_name == "ERANGE"


@pytest.mark.parametrize("dims", DIMS + [(1, 1, 1)])
@pytest.mark.parametrize("n", [1, 2, 4097, 70_001])
def test_lean_build_gives_the_same_arrays(dims, n):
    """The sort that carries positions (the work space of a build that ran out of memory) against the one that carries
    values, with duplicates and with an index out of range."""
    rng = np.random.default_rng(n + sum(dims))
    c = [torch.from_numpy(rng.integers(0, d, n).astype(np.int32)).cuda() for d in dims]
    v = torch.from_numpy(rng.uniform(-1, 1, n)).cuda()
    print("[case] lean build, dims %s n %d" % (dims, n), flush=True)
    one, two = (cst.build_csf(c, v, dims, [1, 2, 0], flags=cst.COALESCE_DUPS | f) for f in (0, cst.LEAN_BUILD))
    for l in range(3):
        for a, b in zip(one.export(l), two.export(l)):
            assert (a is None and b is None) or torch.equal(a, b)
    c[2][n - 1] = dims[2]
    with pytest.raises(Exception, match="below its mode extent"):
        cst.build_csf(c, v, dims, [1, 2, 0], flags=cst.COALESCE_DUPS | cst.LEAN_BUILD)


def test_lean_build_needs_less_work_space():
    n = 30_000_000
    c = [torch.randint(0, 1 << 30, (n,), device="cuda", dtype=torch.int32) for _ in range(2)]
    v = torch.rand(n, dtype=torch.float64, device="cuda")
    print("[case] work space of a build of %d nonzeros" % n, flush=True)
    alive = cst.build_csf([x[:1] for x in c], v[:1], (1 << 30, 1 << 30), [0, 1])
    spent = []
    for flags in (0, cst.LEAN_BUILD):
        cst.release_memory()
        before = torch.cuda.mem_get_info()[0]
        csf = cst.build_csf(c, v, (1 << 30, 1 << 30), [0, 1], flags=cst.COALESCE_DUPS | flags)
        spent.append(before - torch.cuda.mem_get_info()[0])        # the CSF, and the work space kept for reuse
        csf.destroy()
    alive.check()
    assert spent[0] - spent[1] >= 7.5 * n, spent
