"""Three-tensor network on the tiled kernel where W holds something in only some of the blocks of sixteen l: numbers
of such blocks on both sides of a round (8) and of a mask batch (64), another set under every k, against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2401_04836_amd as cst
from paper_2401_04836_amd import schedules as S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("blocks", [1, 7, 8, 9, 63, 64, 65, 129])
@pytest.mark.parametrize("slices", [5, 170])
def test_only_some_blocks_of_l(blocks, slices):
    rng = np.random.default_rng(blocks + slices)
    J, K, L, M = 45, 5, 16 * 131 - 3, 50
    keys = np.unique(rng.integers(0, slices * J * K, slices * 60))
    u = [x.astype(np.int32) for x in np.unravel_index(keys, (slices, J, K))]
    wk, wl = [], []
    for k in range(K - 1):                                # nothing below the last k, fewer blocks below the first
        for b in rng.permutation(131)[:blocks if k else 1 + blocks // 2]:
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
    for waves in (2, 1):
        pl = cst.plan(S.SPTN3, [("U", U), ("V", v), ("W", W)], options=dict(sptn3_tiled=2, sptn3_waves=waves))
        got = cst.execute(pl, [v]).cpu().numpy().reshape(want.shape)
        # at most 45 x 5 x 131 x 4 products of three factors to a sum, in any order: 23582 roundings of 1.1e-16
        assert oracle.rel_err(got, want, S_abs) <= 2.7e-12
