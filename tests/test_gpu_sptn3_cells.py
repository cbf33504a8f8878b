"""Three-tensor network on the tiled kernels where W holds something in only some of the blocks of sixteen l: numbers of such
blocks on both sides of a round (16) and of what a wavefront holds of them (128), whole and in two parts, another set under
every k; and where a wavefront has all the W tiles of a round that it can have (16 blocks of 7 or 4); against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2401_04836_amd as cst
from paper_2401_04836_amd import schedules as S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("blocks", [1, 7, 8, 9, 15, 16, 17, 30, 31, 32, 33, 34, 63, 64, 65, 127, 128, 129, 254, 256, 258])
@pytest.mark.parametrize("slices", [5, 170])
def test_only_some_blocks_of_l(blocks, slices):
    rng = np.random.default_rng(blocks + slices)
    J, K, LT, M = 45, 5, 259, 50
    L = 16 * LT - 3
    keys = np.unique(rng.integers(0, slices * J * K, slices * 60))
    u = [x.astype(np.int32) for x in np.unravel_index(keys, (slices, J, K))]
    wk, wl = [], []
    for k in range(K - 1):                                # nothing below the last k, fewer blocks below the first
        for b in rng.permutation(LT)[:blocks if k else 1 + blocks // 2]:
            n = rng.integers(1, 5)
            wk += [k] * n
            wl += list(np.minimum(16 * b + rng.permutation(16)[:n], L - 1))
    wkey = np.unique((np.repeat(np.array(wk), 4) * L + np.repeat(np.array(wl), 4)) * M + rng.integers(0, M, 4 * len(wk)))
    wc = [x.astype(np.int32) for x in np.unravel_index(wkey, (K, L, M))]
    uv, wv, V = rng.uniform(-1, 1, len(keys)), rng.uniform(-1, 1, len(wkey)), rng.uniform(-1, 1, (J, L))
    print("[case] blocks %d slices %d nnz %d %d" % (blocks, slices, len(uv), len(wv)), flush=True)
    up = lambda cs: [torch.from_numpy(x).cuda() for x in cs]
    U = cst.build_csf(up(u), torch.from_numpy(uv).cuda(), (slices, J, K), [0, 2, 1])
    W = cst.build_csf(up(wc), torch.from_numpy(wv).cuda(), (K, L, M), [0, 1, 2])
    v = torch.from_numpy(V).cuda()
    want = oracle.sptn3(u, uv, (slices, J, K), V, wc, wv, (K, L, M))
    S_abs = oracle.sptn3_abs(u, uv, (slices, J, K), V, wc, wv, (K, L, M))
    # one chunk of the k range takes the blocks whole; several chunks of few groups take them in two parts
    for waves, cut, wgs in ((2, 32, 8000), (2, 32, 1), (2, 16, 8000), (2, 16, 1), (1, 0, 8000)):
        pl = cst.plan(S.SPTN3, [("U", U), ("V", v), ("W", W)],
                      options=dict(sptn3_tiled=2, sptn3_waves=waves, sptn3_slices=cut, sptn3_wgs=wgs))
        got = cst.execute(pl, [v]).cpu().numpy().reshape(want.shape)
        # at most 45 x 5 x 259 x 4 products of three factors to a sum, in any order: 46624 roundings of 1.1e-16
        assert oracle.rel_err(got, want, S_abs) <= 5.2e-12


@pytest.mark.parametrize("M", [400, 399, 385, 224])
@pytest.mark.parametrize("L", [256, 275])
def test_every_w_tile_of_a_round(L, M):
    """A dense W: 25 m tiles below every block of l, so that a wavefront's list of a round holds up to 112 places."""
    rng = np.random.default_rng(L + M)
    slices, J, K = 40, 30, 3
    keys = np.unique(rng.integers(0, slices * J * K, 1500))
    u = [x.astype(np.int32) for x in np.unravel_index(keys, (slices, J, K))]
    wc = [x.ravel().astype(np.int32) for x in np.meshgrid(np.arange(K), np.arange(L), np.arange(M), indexing="ij")]
    uv, wv, V = rng.uniform(-1, 1, len(keys)), rng.uniform(-1, 1, wc[0].size), rng.uniform(-1, 1, (J, L))
    print("[case] dense W, L %d M %d" % (L, M), flush=True)
    up = lambda cs: [torch.from_numpy(x).cuda() for x in cs]
    U = cst.build_csf(up(u), torch.from_numpy(uv).cuda(), (slices, J, K), [0, 2, 1])
    W = cst.build_csf(up(wc), torch.from_numpy(wv).cuda(), (K, L, M), [0, 1, 2])
    v = torch.from_numpy(V).cuda()
    want = oracle.sptn3(u, uv, (slices, J, K), V, wc, wv, (K, L, M))
    S_abs = oracle.sptn3_abs(u, uv, (slices, J, K), V, wc, wv, (K, L, M))
    for waves, cut in ((2, 32), (2, 16), (1, 0)):
        pl = cst.plan(S.SPTN3, [("U", U), ("V", v), ("W", W)], options=dict(sptn3_waves=waves, sptn3_slices=cut))
        assert "tiled" in pl.describe()
        got = cst.execute(pl, [v]).cpu().numpy().reshape(want.shape)
        # (J + K L + 3) roundings along the longest chain of a sum
        assert oracle.rel_err(got, want, S_abs) <= (J + K * L + 3) * 1.1e-16
