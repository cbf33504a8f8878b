"""Three-tensor network on the kernel with two wavefronts per SIMD, in groups of 32 slices and of 16: numbers of slices on both sides of a half (16) and of a
group (32), unions of j on both sides of a batch (8), of a group of batches (32) and of a pass (312), odd and even numbers of mask
words (J = 31, 70, 2000; 33, 640), rows of the union that only one half holds, few pairs over many blocks of l (each pair takes half of them), slices and pairs without work, against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2401_04836_amd as cst
from paper_2401_04836_amd import schedules as S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("wgs", [1, 8000])
@pytest.mark.parametrize("slices,J,shared", [(1, 1, True), (16, 8, True), (17, 33, False), (32, 312, True), (33, 313, False),
                                             (40, 640, False), (65, 31, True), (20, 70, False), (18, 2000, False)])
@pytest.mark.parametrize("L", [40, 600])
def test_halves_passes_and_parts(slices, J, shared, L, wgs):
    rng = np.random.default_rng(slices * 1000 + J + L)
    K, M, rows = 7, 70, slices + 5                        # five rows of the result have no slice
    row_of = np.sort(rng.permutation(rows)[:slices])
    per_half = max(1, J // 2)                             # not shared: halves hold different j, a few of them in common
    u = [[], [], []]
    for s in range(slices):
        for k in range(K - 1):                            # no slice holds the last k
            if k == 2 and s >= 16:
                continue                                  # here the first half alone
            js = np.arange(J) if shared else np.unique(np.concatenate([np.arange(per_half) + (s // 16 % 2) * (J - per_half),
                                                                       rng.integers(0, J, 2)]))
            js = js[rng.random(js.size) < 0.9] if js.size > 1 else js
            u[0] += [row_of[s]] * js.size
            u[1] += list(js)
            u[2] += [k] * js.size
    u = [np.array(x, dtype=np.int32) for x in u]
    wkey = np.unique(rng.integers(0, 5 * L * M, 6 * L))   # nothing in W below the fifth k and on
    wc = [x.astype(np.int32) for x in np.unravel_index(wkey, (K, L, M))]
    uv, wv, V = rng.uniform(-1, 1, u[0].size), rng.uniform(-1, 1, wkey.size), rng.uniform(-1, 1, (J, L))
    print("[case] slices %d J %d shared %s L %d wgs %d nnz %d %d" % (slices, J, shared, L, wgs, uv.size, wv.size), flush=True)
    up = lambda cs: [torch.from_numpy(x).cuda() for x in cs]
    U = cst.build_csf(up(u), torch.from_numpy(uv).cuda(), (rows, J, K), [0, 2, 1])
    W = cst.build_csf(up(wc), torch.from_numpy(wv).cuda(), (K, L, M), [0, 1, 2])
    v = torch.from_numpy(V).cuda()
    want = oracle.sptn3(u, uv, (rows, J, K), V, wc, wv, (K, L, M))
    S_abs = oracle.sptn3_abs(u, uv, (rows, J, K), V, wc, wv, (K, L, M))
    for flags, cut in ((0, 32), (cst.OUT_COMPACT, 32), (0, 16), (cst.OUT_COMPACT, 16)):
        pl = cst.plan(S.SPTN3, [("U", U), ("V", v), ("W", W)], flags=flags, options=dict(sptn3_tiled=2, sptn3_wgs=wgs, sptn3_slices=cut))
        assert "two waves" in pl.describe() and "slices %d" % cut in pl.describe()
        got = cst.execute(pl, [v]).cpu().numpy().reshape(-1, M)
        ref, bound = (want[row_of], S_abs[row_of]) if flags else (want, S_abs)
        assert not np.isnan(got).any() and not got[bound == 0].any()
        # a sum has at most J K x L products of three factors, in any order: (J + K L + 3) roundings along the longest chain
        assert oracle.rel_err(got, ref, bound) <= (J + K * L + 3) * 1.1e-16


@pytest.mark.parametrize("cut,waves", [(32, 2), (16, 2), (0, 1)])
def test_more_elements_than_a_launch_has_threads_for(cut, waves):
    """A root mode of 10.8 M indices, of which forty hold anything, times 400: 2^32 elements and more, 35 GB.  Every row is
    written, those without a slice with zeros."""
    rows, M, J, K, L = (1 << 32) // 400 + 40_000, 400, 9, 5, 40
    if torch.cuda.mem_get_info()[0] < 8 * rows * M + (4 << 30):
        pytest.skip("the result does not fit the free device memory")
    rng = np.random.default_rng(9200)
    at = np.sort(rng.choice(rows, 40, replace=False))
    at[-1] = rows - 1
    ukey = np.unique(rng.integers(0, 40 * J * K, 900))
    u = [x.astype(np.int32) for x in np.unravel_index(ukey, (40, J, K))]
    wkey = np.unique(rng.integers(0, K * L * M, 3000))
    wc = [x.astype(np.int32) for x in np.unravel_index(wkey, (K, L, M))]
    uv, wv, V = rng.uniform(-1, 1, len(ukey)), rng.uniform(-1, 1, len(wkey)), rng.uniform(-1, 1, (J, L))
    print("[case] %d rows of %d, waves %d, slices %d" % (rows, M, waves, cut), flush=True)
    up = lambda cs: [torch.from_numpy(x).cuda() for x in cs]
    U = cst.build_csf(up([at[u[0]].astype(np.int32), u[1], u[2]]), torch.from_numpy(uv).cuda(), (rows, J, K), [0, 2, 1])
    W = cst.build_csf(up(wc), torch.from_numpy(wv).cuda(), (K, L, M), [0, 1, 2])
    v = torch.from_numpy(V).cuda()
    want = oracle.sptn3(u, uv, (40, J, K), V, wc, wv, (K, L, M))
    S_abs = oracle.sptn3_abs(u, uv, (40, J, K), V, wc, wv, (K, L, M))
    pl = cst.plan(S.SPTN3, [("U", U), ("V", v), ("W", W)], options=dict(sptn3_tiled=2, sptn3_waves=waves, sptn3_slices=cut))
    assert "k chunks 1 " not in pl.describe() + " "
    out = torch.full((rows * M,), 7.0, dtype=torch.float64, device="cuda")
    cst.execute(pl, [v], out=out)
    got = out.view(rows, M)[torch.from_numpy(at).cuda()].cpu().numpy()
    nonzero = sum(int(torch.count_nonzero(part)) for part in out.split(1 << 28))
    del out
    torch.cuda.empty_cache()
    # a sum has at most J K x L products of three factors, in any order: (J + K L + 3) roundings along the longest chain
    assert oracle.rel_err(got, want, S_abs) <= (J + K * L + 3) * 1.1e-16
    assert nonzero == np.count_nonzero(want)


@pytest.mark.parametrize("slices,J,K,cut", [(20, 60, 6, 16), (4096, 8, 64, 32)])
def test_slices_of_a_group_follow_the_pairs_of_the_chip(slices, J, K, cut):
    """Groups of 16 where a compute unit has one pair or none, of 32 where it has many; both forms give the same sums."""
    rng = np.random.default_rng(slices)
    L, M = 64, 48
    u = [x.ravel().astype(np.int32) for x in np.meshgrid(np.arange(slices), np.arange(J), np.arange(K), indexing="ij")]
    wc = [x.ravel().astype(np.int32) for x in np.meshgrid(np.arange(K), np.arange(L), np.arange(M), indexing="ij")]
    uv, wv, V = rng.uniform(-1, 1, u[0].size), rng.uniform(-1, 1, wc[0].size), rng.uniform(-1, 1, (J, L))
    print("[case] %d slices, J %d, K %d" % (slices, J, K), flush=True)
    up = lambda cs: [torch.from_numpy(x).cuda() for x in cs]
    U = cst.build_csf(up(u), torch.from_numpy(uv).cuda(), (slices, J, K), [0, 2, 1])
    W = cst.build_csf(up(wc), torch.from_numpy(wv).cuda(), (K, L, M), [0, 1, 2])
    v = torch.from_numpy(V).cuda()
    want = np.tensordot(np.tensordot(uv.reshape(slices, J, K), V, (1, 0)), wv.reshape(K, L, M), ((1, 2), (0, 1)))
    a, b, c = (np.abs(x) for x in (uv.reshape(slices, J, K), V, wv.reshape(K, L, M)))
    S_abs = np.tensordot(np.tensordot(a, b, (1, 0)), c, ((1, 2), (0, 1)))
    for told in (0, 16, 32):
        pl = cst.plan(S.SPTN3, [("U", U), ("V", v), ("W", W)], options=dict(sptn3_slices=told))
        assert "slices %d" % (told or cut) in pl.describe()
        got = cst.execute(pl, [v]).cpu().numpy().reshape(slices, M)
        # (J + K L + 3) roundings along the longest chain, on both sides
        assert oracle.rel_err(got, want, S_abs) <= 2 * (J + K * L + 3) * 1.1e-16


def test_a_compute_unit_that_another_stream_holds():
    """Several pairs per compute unit, one of which another stream holds for many times the network's time: its share goes to
    the others (an eighth more for each of them here), it does not wait for a second round of the whole."""
    rng = np.random.default_rng(9300)
    slices, J, K, L, M = 1024, 64, 64, 512, 64
    u = [x.ravel().astype(np.int32) for x in np.meshgrid(np.arange(slices), np.arange(J), np.arange(K), indexing="ij")]
    wc = [x.ravel().astype(np.int32) for x in np.meshgrid(np.arange(K), np.arange(L), np.arange(M), indexing="ij")]
    up = lambda x: torch.from_numpy(x).cuda()
    U = cst.build_csf([up(x) for x in u], up(rng.uniform(-1, 1, u[0].size)), (slices, J, K), [0, 2, 1])
    W = cst.build_csf([up(x) for x in wc], up(rng.uniform(-1, 1, wc[0].size)), (K, L, M), [0, 1, 2])
    v = up(rng.uniform(-1, 1, (J, L)))
    pl = cst.plan(S.SPTN3, [("U", U), ("V", v), ("W", W)])
    out = torch.empty(slices * M, dtype=torch.float64, device="cuda")
    side, event = torch.cuda.Stream(), lambda: torch.cuda.Event(enable_timing=True)

    def best_ms(f):
        times = []
        for _ in range(5):
            torch.cuda.synchronize()
            a, b = event(), event()
            f(a, b)
            torch.cuda.synchronize()
            times.append(a.elapsed_time(b))
        return min(times)

    def network(a, b):
        a.record()
        cst.execute(pl, [v], out=out)
        b.record()

    def sleep(a, b):
        a.record()
        torch.cuda._sleep(1_000_000)
        b.record()

    def held(a, b):
        with torch.cuda.stream(side):
            torch.cuda._sleep(cycles)
            begun.record()
        network(a, b)

    begun = event()
    alone, per_cycle = best_ms(network), best_ms(sleep) / 1_000_000
    cycles = int(20 * alone / per_cycle)                       # one workgroup of one wavefront, 20 times as long
    beside = best_ms(held)
    print("[case] alone %.3f ms, beside a held compute unit %.3f ms" % (alone, beside), flush=True)
    assert beside < 1.5 * alone
