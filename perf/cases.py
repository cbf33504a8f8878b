"""Timed cases of the library: what a program that contracts sparse tensors calls, over the sizes it calls it with.

Every case is one pass through the three verbs: `build_csf` (coordinates to CSF), or `execute` of a plan that
the program keeps beside its tensor while the dense factors change.  Kinds:

    build      COO -> CSF of an order-3 or order-4 tensor, once per new tensor
    mttkrp3    order-3 MTTKRP of one output mode (one step of a CP-ALS sweep)
    mttkrp4    order-4 MTTKRP, the same at the next order up
    ttmc3      order-3 TTMc (one step of a Tucker/HOOI sweep), dense rows or rows of nonempty slices only
    ttmc4      order-4 TTMc
    sptn3      the three-tensor network Z = (U.V).W with block-sparse U and W
    spchain3   the sparse three-index integral transformation E = I.C.P on lattice maps, with or without filter
    sppair4    the four-index product V = E.E of its result

Inputs are synthetic: coordinates uniform or Zipf-distributed over shuffled indices and made distinct, values
uniform or normal, everything drawn on the GPU from the seed.
"""
import math

import numpy as np
import torch

import paper_2401_04836_amd as cst
from paper_2401_04836_amd import schedules

MTTKRP4 = ("T1[i,j,k,r] = X[i,j,k,l] * D[l,r] | i,j,k,l,r ; T2[i,j,r] = T1[i,j,k,r] * C[k,r] | i,j,k,r ; "
           "M[i,r] = T2[i,j,r] * B[j,r] | i,j,r")


def listed():
    return [
        # a tensor that fits any cache: the launch and the host path are the time
        dict(name="ttmc3_tiny_r8", kind="ttmc3", i=200, j=200, k=200, s_i=0.0, s_j=0.0, s_k=0.0,
             nnz=8_000, r2=8, r3=8, compact=False),
        # one mode of a CP step on a small log of events: fewer leaves than lanes of the chip
        dict(name="mttkrp3_small_r32", kind="mttkrp3", i=1203, j=907, k=2903, s=1.1, nnz=150_001, rank=32, mode=2),
        # CP of a tagged-items tensor at rank 50 (the rank of Sec. 5.2), output mode in the middle
        dict(name="mttkrp3_mid_r50", kind="mttkrp3", i=320_011, j=28_201, k=16_007, s=1.05, nnz=20_000_003, rank=50,
             mode=1),
        # the largest MTTKRP of the benchmark
        dict(name="mttkrp3_76m_r32", kind="mttkrp3", i=12_000, j=9_000, k=29_000, s=1.1, nnz=76_000_000, rank=32,
             mode=0),
        # CP of an order-4 tensor
        dict(name="mttkrp4_20m_r32", kind="mttkrp4", i=1_000, j=50_000, k=50_000, l=2_000, s=1.05, nnz=20_000_000,
             rank=32),
        # Tucker at rank 50 (Sec. 5.3): no multiple of a matrix tile
        dict(name="ttmc3_mid_r50", kind="ttmc3", i=12_007, j=9_001, k=28_999, s_i=1.1, s_j=1.1, s_k=1.1,
             nnz=5_000_011, r2=50, r3=50, compact=False),
        # Tucker at the largest tuned ranks on a strongly skewed tensor, rows of nonempty slices only
        dict(name="ttmc3_skew_r64", kind="ttmc3", i=200_003, j=300_007, k=25_000, s_i=1.3, s_j=1.3, s_k=0.0,
             nnz=14_000_000, r2=64, r3=64, compact=True),
        # order-4 Tucker of the benchmark
        dict(name="ttmc4_40m_r16", kind="ttmc4", i=1_000, j=50_000, k=50_000, l=2_000, s=1.05, nnz=40_000_000,
             r1=16, r2=16, r3=16),
        # the three-tensor network of the benchmark: blocks of 100 x 100 x 20
        dict(name="sptn3_block", kind="sptn3", i=2000, j=2000, k=400, l=2000, m=400, nb=20, sel_u=640, sel_w=800),
        # three-index transformation on a 32 x 32 lattice
        dict(name="spchain3_32", kind="spchain3", side=32, n_ao=3, n_df=14, restricted=False),
        # four-index product on a 12 x 12 lattice
        dict(name="sppair4_12", kind="sppair4", side=12, n_ao=3, n_df=10),
        # a new tensor of the largest MTTKRP's size arrives
        dict(name="build_76m", kind="build", i=12_000, j=9_000, k=29_000, l=0, s=1.1, nnz=76_000_000, first=0),
    ]


def _log(rng, lo, hi):
    """An integer between lo and hi, spread over the logarithm."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["build", "mttkrp3", "mttkrp3", "mttkrp3", "mttkrp4", "ttmc3", "ttmc3", "ttmc3", "ttmc4",
                       "sptn3", "spchain3", "sppair4"])
    if kind == "build":
        c = dict(kind=kind, i=_log(rng, 1_000, 500_000), j=_log(rng, 1_000, 100_000), k=_log(rng, 1_000, 100_000),
                 l=rng.choice([0, 0, 500, 2003]), s=rng.choice([0.0, 1.05, 1.1]), nnz=_log(rng, 8_000, 60_000_000),
                 first=rng.randrange(3))
    elif kind == "mttkrp3":
        c = dict(kind=kind, i=_log(rng, 1_000, 500_000), j=_log(rng, 900, 50_000), k=_log(rng, 1_000, 50_000),
                 s=rng.choice([0.0, 1.05, 1.1]), nnz=_log(rng, 20_000, 40_000_000),
                 rank=rng.choice([8, 10, 16, 25, 32, 32, 50, 64, 100]), mode=rng.randrange(3))
        if c["nnz"] * c["rank"] > 76_000_000 * 32:
            c["nnz"] = 76_000_000 * 32 // c["rank"]
    elif kind == "mttkrp4":
        c = dict(kind=kind, i=_log(rng, 500, 20_000), j=_log(rng, 2_000, 50_000), k=_log(rng, 2_000, 50_000),
                 l=_log(rng, 500, 5_000), s=rng.choice([0.0, 1.05]), nnz=_log(rng, 50_000, 20_000_000),
                 rank=rng.choice([8, 16, 25, 32, 50]))
    elif kind == "ttmc3":
        r2, r3 = (rng.choice([8, 10, 16, 20, 32, 50, 64]) for _ in range(2))
        c = dict(kind=kind, i=_log(rng, 200, 100_000), j=_log(rng, 200, 200_000), k=_log(rng, 200, 30_000),
                 s_i=rng.choice([0.0, 1.1, 1.3]), s_j=rng.choice([0.0, 1.1, 1.3]), s_k=rng.choice([0.0, 1.1]),
                 nnz=_log(rng, 8_000, 8_000_000), r2=r2, r3=r3, compact=rng.random() < 0.5)
    elif kind == "ttmc4":
        r = rng.choice([(16, 16, 16), (16, 16, 16), (8, 8, 8), (10, 12, 7)])
        c = dict(kind=kind, i=_log(rng, 100, 3_000), j=_log(rng, 1_000, 50_000), k=_log(rng, 1_000, 50_000),
                 l=_log(rng, 200, 2_000), s=rng.choice([0.0, 1.05]), nnz=_log(rng, 50_000, 8_000_000),
                 r1=r[0], r2=r[1], r3=r[2])
    elif kind == "sptn3":
        nb = rng.choice([4, 10, 16, 20])
        b = [rng.randrange(lo, hi + 1) for lo, hi in ((8, 90), (8, 90), (3, 20), (8, 90), (8, 20))]
        c = dict(kind=kind, i=nb * b[0], j=nb * b[1], k=nb * b[2], l=nb * b[3], m=nb * b[4], nb=nb,
                 sel_u=max(2, int(nb ** 3 * rng.uniform(0.03, 0.1))), sel_w=max(2, int(nb ** 3 * rng.uniform(0.05, 0.1))))
    elif kind == "spchain3":
        c = dict(kind=kind, side=rng.randrange(8, 33), n_ao=3, n_df=rng.randrange(6, 15), restricted=rng.random() < 0.5)
    else:
        c = dict(kind=kind, side=rng.randrange(5, 13), n_ao=3, n_df=rng.randrange(6, 11))
    if "nnz" in c:                                   # distinct coordinates stay easy to find
        cells = c["i"] * c["j"] * c["k"] * max(1, c.get("l", 1))
        c["nnz"] = min(c["nnz"], cells // 50 + 100)
    return c


# ---- inputs -------------------------------------------------------------------------------------------------


def _dev():
    return torch.device("cuda", torch.cuda.current_device())


def _uniform(g, *shape, lo=-1.0, hi=1.0):
    return torch.rand(*shape, generator=g, dtype=torch.float64, device=g.device) * (hi - lo) + lo


def _normal(g, *shape):
    return torch.randn(*shape, generator=g, dtype=torch.float64, device=g.device)


def _weights(n, s):
    """Probabilities of the n indices of a mode, most frequent first."""
    w = np.arange(1, n + 1, dtype=np.float64) ** (-float(s))
    return w / w.sum()


TEMPLATE = 20240104        # seed of the structures that the inputs' own seeds relabel


def _ranks(g, n, s, count):
    """Frequency ranks of `count` draws from a mode of extent n: uniform (s = 0) or P(rank r) ~ r**-s."""
    if not s:
        return torch.randint(n, (count,), generator=g, device=g.device)
    cdf = torch.from_numpy(np.cumsum(_weights(n, s))).to(g.device)
    u = torch.rand(count, generator=g, dtype=torch.float64, device=g.device)
    return torch.clamp(torch.searchsorted(cdf, u, right=True), max=n - 1)


def _relabelled(g, ranks, dims):
    """int32 coordinates: the indices of every mode renamed, the nonzeros in another order."""
    order = torch.randperm(ranks[0].numel(), generator=g, device=g.device)
    return [torch.randperm(n, generator=g, device=g.device)[r[order]].to(torch.int32) for r, n in zip(ranks, dims)]


def _coords(g, dims, skews, nnz):
    """nnz distinct coordinate tuples in random order: one int32 tensor per mode.  Inputs of two seeds differ in
    every index and in the order of the nonzeros, and have the same numbers of slices and fibers."""
    t = torch.Generator(device=g.device).manual_seed(TEMPLATE)
    keys = torch.empty(0, dtype=torch.int64, device=g.device)
    while keys.numel() < nnz:
        need = nnz - keys.numel()
        batch = need + need // 3 + 1024
        key = torch.zeros(batch, dtype=torch.int64, device=g.device)
        for n, s in zip(dims, skews):
            key = key * n + _ranks(t, n, s, batch)
        keys = torch.unique(torch.cat([keys, key]))
    keys = keys[torch.randperm(keys.numel(), generator=t, device=g.device)[:nnz]]
    ranks = []
    for n in reversed(dims):
        ranks.append(keys % n)
        keys = keys // n
    return _relabelled(g, ranks[::-1], dims)


def _block_sparse(g, dims, nb, selected):
    """A grid of nb blocks per mode, `selected` of them dense inside; coordinates block by block."""
    size = [d // nb for d in dims]
    blocks = torch.randperm(nb ** len(dims), generator=g, device=g.device)[:selected]
    volume = math.prod(size)
    e = torch.arange(selected * volume, dtype=torch.int64, device=g.device)
    block, inner = blocks[e // volume], e % volume
    out = []
    for s in reversed(size):
        out.append(((block % nb) * s + inner % s).to(torch.int32))
        block, inner = block // nb, inner // s
    return out[::-1]


R_INT, R_MO, R_PAO, R_FILTER = 2.0, 2.0, 2.0, 3.0        # cut-off radii of the lattice maps
KEEP_INT, KEEP_MO, KEEP_PAO = 0.7, 0.85, 0.85            # share of the entries within them that is stored


def _near(side, radius, device):
    """near[a, b]: atoms a and b of a side x side lattice lie within `radius`."""
    a = torch.arange(side * side, device=device)
    x, y = a // side, a % side
    return ((x[:, None] - x[None]) ** 2 + (y[:, None] - y[None]) ** 2) <= radius * radius


def _pairs(t, near, na, nb, keep):
    """Pairs of functions (na on the first atom, nb on the second) on near atoms, a share `keep` of them."""
    pa, pb = near.nonzero(as_tuple=True)
    f = torch.arange(na * nb, device=t.device)
    ca = (pa[:, None] * na + f // nb).reshape(-1)
    cb = (pb[:, None] * nb + f % nb).reshape(-1)
    k = torch.rand(ca.numel(), generator=t, device=t.device) < keep
    return [ca[k], cb[k]]


def _turned(g, side):
    """One of the lattice's eight symmetries: the new label of every atom."""
    a = torch.arange(side * side, device=g.device).reshape(side, side)
    turn, flip = (int(torch.randint(n, (1,), generator=g, device=g.device)) for n in (4, 2))
    a = torch.rot90(a, turn)
    return (a.flip(0) if flip else a).reshape(-1)


def _names(g, atom, n):
    """New label of every function, n on an atom: those of one atom in another order, on the atom's new place."""
    inside = torch.rand(atom.numel(), n, generator=g, device=g.device).argsort(1)
    return (atom[:, None] * n + inside).reshape(-1)


def _lattice(g, side, n_ao, n_df, restricted):
    """Operands of the chain as CSF handles: I K>u>v, C i>u, P m>v and the filter L K>i.  Inputs of two seeds differ
    in the atoms' places, the functions' order and every value, and have results of one size."""
    dev, atoms = g.device, side * side
    t = torch.Generator(device=dev).manual_seed(TEMPLATE)
    near = _near(side, R_INT, dev)
    k, u = near.nonzero(as_tuple=True)
    row, v = (near[k] & near[u]).nonzero(as_tuple=True)
    k, u = k[row], u[row]
    f = torch.arange(n_df * n_ao * n_ao, device=dev)
    coords = [(k[:, None] * n_df + f // (n_ao * n_ao)).reshape(-1), (u[:, None] * n_ao + f // n_ao % n_ao).reshape(-1),
              (v[:, None] * n_ao + f % n_ao).reshape(-1)]
    keep = torch.rand(coords[0].numel(), generator=t, device=dev) < KEEP_INT
    coords = [c[keep] for c in coords]
    n_K, n_i, n_u = atoms * n_df, atoms, atoms * n_ao
    atom = _turned(g, side)
    K, i, ao, m = _names(g, atom, n_df), _names(g, atom, 1), _names(g, atom, n_ao), _names(g, atom, n_ao)

    def csf(coords, labels, dims, mode_order, ones=False):
        coords = [label[c].to(torch.int32) for c, label in zip(coords, labels)]
        n = coords[0].numel()
        vals = torch.ones(n, dtype=torch.float64, device=dev) if ones else _normal(g, n)
        return cst.build_csf(coords, vals, dims, mode_order)

    ops = [("I", csf(coords, (K, ao, ao), (n_K, n_u, n_u), [0, 1, 2])),
           ("C", csf(_pairs(t, _near(side, R_MO, dev), n_ao, 1, KEEP_MO), (ao, i), (n_u, n_i), [1, 0]))]
    if restricted:
        ops.append(("L", csf(_pairs(t, _near(side, R_FILTER, dev), n_df, 1, 1.0), (K, i), (n_K, n_i), [0, 1], ones=True)))
    ops.append(("P", csf(_pairs(t, _near(side, R_PAO, dev), n_ao, n_ao, KEEP_PAO), (ao, m), (n_u, n_u), [1, 0])))
    return ops


def prepare(case, seed):
    kind = case["kind"]
    g = torch.Generator(device=_dev()).manual_seed(seed)
    state = dict(case=case)
    if kind == "build":
        dims = [case[m] for m in "ijkl" if case[m]]
        state["coords"] = _coords(g, dims, [case["s"]] * len(dims), case["nnz"])
        state["vals"] = _uniform(g, case["nnz"], lo=0.0)
        state["dims"] = dims
        state["mode_order"] = [(case["first"] + m) % len(dims) for m in range(len(dims))]
    elif kind == "mttkrp3":
        dims = [case[m] for m in "ijk"]
        coords = _coords(g, dims, [case["s"]] * 3, case["nnz"])
        levels = [case["mode"]] + [m for m in range(3) if m != case["mode"]]
        csf = cst.build_csf(coords, _uniform(g, case["nnz"], lo=0.0), dims, levels)
        text, names = schedules.mttkrp3_for(levels)
        leaf, middle = _uniform(g, dims[levels[2]], case["rank"]), _uniform(g, dims[levels[1]], case["rank"])
        state["plan"] = cst.plan(text, [("X", csf), (names[1], leaf), (names[2], middle)])
        state["factors"] = [leaf, middle]
    elif kind == "mttkrp4":
        dims = [case[m] for m in "ijkl"]
        coords = _coords(g, dims, [0.0] + [case["s"]] * 3, case["nnz"])
        csf = cst.build_csf(coords, _normal(g, case["nnz"]), dims, [0, 1, 2, 3])
        B, C, D = (_uniform(g, d, case["rank"]) for d in dims[1:])
        state["plan"] = cst.plan(MTTKRP4, [("X", csf), ("D", D), ("C", C), ("B", B)])
        state["factors"] = [D, C, B]
    elif kind == "ttmc3":
        dims = [case[m] for m in "ijk"]
        coords = _coords(g, dims, [case["s_i"], case["s_j"], case["s_k"]], case["nnz"])
        csf = cst.build_csf(coords, _uniform(g, case["nnz"]), dims, [0, 1, 2])
        U2, U3 = _uniform(g, dims[1], case["r2"]), _uniform(g, dims[2], case["r3"])
        state["plan"] = cst.plan(schedules.TTMC3, [("X", csf), ("U3", U3), ("U2", U2)],
                                 flags=cst.OUT_COMPACT if case["compact"] else 0)
        state["factors"] = [U3, U2]
    elif kind == "ttmc4":
        dims = [case[m] for m in "ijkl"]
        coords = _coords(g, dims, [0.0] + [case["s"]] * 3, case["nnz"])
        csf = cst.build_csf(coords, _normal(g, case["nnz"]), dims, [0, 1, 2, 3])
        U1, U2, U3 = _normal(g, dims[1], case["r1"]), _normal(g, dims[2], case["r2"]), _normal(g, dims[3], case["r3"])
        state["plan"] = cst.plan(schedules.TTMC4, [("X", csf), ("U3", U3), ("U2", U2), ("U1", U1)])
        state["factors"] = [U3, U2, U1]
    elif kind == "sptn3":
        I, J, K, L, M = (case[x] for x in "ijklm")
        u = _block_sparse(g, (I, J, K), case["nb"], case["sel_u"])
        w = _block_sparse(g, (K, L, M), case["nb"], case["sel_w"])
        U = cst.build_csf(u, _normal(g, u[0].numel()), (I, J, K), [0, 2, 1])
        W = cst.build_csf(w, _normal(g, w[0].numel()), (K, L, M), [0, 1, 2])
        V = _normal(g, J, L)
        state["plan"] = cst.plan(schedules.SPTN3, [("U", U), ("V", V), ("W", W)])
        state["factors"] = [V]
    else:
        ops = _lattice(g, case["side"], case["n_ao"], case["n_df"], case.get("restricted", False))
        chain = cst.plan(schedules.SPCHAIN3_RESTRICTED if case.get("restricted") else schedules.SPCHAIN3, ops)
        state["plan"], state["factors"] = chain, []
        if kind == "sppair4":
            values, E = cst.execute(chain, []), chain.output_csf()
            (iK, pK, _), (ii, pi, _), (im, _, _) = E.export(0), E.export(1), E.export(2)
            n = pi[1:] - pi[:-1]
            K = torch.repeat_interleave(torch.repeat_interleave(iK, pK[1:] - pK[:-1]), n)
            atoms = case["side"] ** 2
            handle = cst.build_csf([K, torch.repeat_interleave(ii, n), im], values,
                                   (atoms * case["n_df"], atoms, atoms * case["n_ao"]), [1, 0, 2])
            state["plan"] = cst.plan(schedules.SPPAIR4, [("Ea", handle), ("Eb", handle)])
    return state


def run(state):
    if state["case"]["kind"] == "build":
        csf = cst.build_csf(state["coords"], state["vals"], state["dims"], state["mode_order"])
        return [csf.export(level) for level in range(csf.order)]
    return cst.execute(state["plan"], state["factors"])


# ---- what a pass cannot do without --------------------------------------------------------------------------


def _bins(n, s, bins=96):
    """(indices in the bin, probability of one of them) for the n indices of a mode, binned by rank."""
    edges = np.unique(np.concatenate([np.arange(min(n, 64) + 1), np.geomspace(1, n, bins).astype(np.int64), [n]]))
    cum = np.concatenate([[0.0], np.cumsum(_weights(n, s))])
    count = np.diff(edges).astype(np.float64)
    return count, np.diff(cum[edges]) / count


def _expected_nodes(dims, skews, nnz):
    """Expected number of distinct coordinate prefixes of nnz draws, per level."""
    out, count, p = [], np.ones(1), np.ones(1)
    for d, (n, s) in enumerate(zip(dims[:-1], skews[:-1])):
        c, q = _bins(n, s)
        count, p = np.outer(count, c).reshape(-1), np.outer(p, q).reshape(-1)
        out.append(min(float(nnz), float((count * -np.expm1(-nnz * p)).sum())))
    return out + [float(nnz)]


def _lattice_sizes(case):
    """Expected stored entries: I, C + P, E, per-K sum of squares of E's rows, V (None for the chain alone)."""
    side, n_ao, n_df = case["side"], case["n_ao"], case["n_df"]
    near = _near(side, R_INT, "cpu").numpy()
    mo, pao = _near(side, R_MO, "cpu").numpy(), _near(side, R_PAO, "cpu").numpy()
    keep = _near(side, R_FILTER, "cpu").numpy()
    atoms = side * side
    n_int, blocks = 0, []
    for K in range(atoms):
        a = np.flatnonzero(near[K])
        pairs = near[np.ix_(a, a)]
        n_int += int(pairs.sum())
        i, m = np.flatnonzero(mo[a].any(0)), np.flatnonzero(pao[a].any(0))
        e = (mo[np.ix_(a, i)].T.astype(np.float32) @ pairs.astype(np.float32) @ pao[np.ix_(a, m)].astype(np.float32)) > 0
        if case.get("restricted"):
            e &= keep[K, i][:, None]
        blocks.append((i, m, e))
    n_E = n_df * n_ao * sum(float(e.sum()) for _, _, e in blocks)
    squares = n_df * sum(float(n_ao * e.sum()) ** 2 for _, _, e in blocks)
    n_V = None
    if case["kind"] == "sppair4":
        at = np.zeros((atoms, atoms * atoms), dtype=bool)
        for K, (i, m, e) in enumerate(blocks):
            at[K, (i[:, None] * atoms + m[None]).reshape(-1)] = e.reshape(-1)
        cols = torch.from_numpy(at[:, at.any(0)].astype(np.float32))
        n_V = float(n_ao ** 2) * sum(float(((cols[:, s:s + 1024].T @ cols) > 0).sum()) for s in range(0, cols.shape[1], 1024))
    return (KEEP_INT * n_int * n_df * n_ao ** 2, KEEP_MO * float(mo.sum()) * n_ao + KEEP_PAO * float(pao.sum()) * n_ao ** 2,
            n_E, squares, n_V)


def work(case):
    """Every CSF entry once (index 4 B and value or child pointer 8 B), every factor once, the output once; the
    multiply-adds of the schedule at the expected number of nodes per level."""
    kind = case["kind"]
    if kind in ("build", "mttkrp3", "mttkrp4", "ttmc3", "ttmc4"):
        dims = [case[m] for m in "ijkl" if case.get(m)]
        if kind == "ttmc3":
            skews = [case["s_i"], case["s_j"], case["s_k"]]
        else:
            skews = [case["s"]] * len(dims)
            if kind in ("mttkrp4", "ttmc4"):
                skews[0] = 0.0
        order = list(range(len(dims)))
        if kind == "build":
            order = [(case["first"] + m) % len(dims) for m in order]
        elif kind == "mttkrp3":
            order = [case["mode"]] + [m for m in order if m != case["mode"]]
        dims, skews = [dims[m] for m in order], [skews[m] for m in order]
        nodes = _expected_nodes(dims, skews, case["nnz"])
        tree = 12.0 * sum(nodes)
        if kind == "build":
            return {"bytes": tree + (4.0 * len(dims) + 8.0) * case["nnz"], "flops": 0.0}
        if kind.startswith("mttkrp"):
            return {"bytes": tree + 8.0 * case["rank"] * sum(dims), "flops": 2.0 * case["rank"] * sum(nodes[1:])}
        ranks = [case[r] for r in ("r1", "r2", "r3") if r in case]
        rows = nodes[0] if case.get("compact") else dims[0]
        flops, width = 0.0, 1
        for level, r in zip(range(len(dims) - 1, 0, -1), reversed(ranks)):
            width *= r
            flops += 2.0 * width * nodes[level]
        return {"bytes": tree + 8.0 * sum(d * r for d, r in zip(dims[1:], ranks)) + 8.0 * rows * width, "flops": flops}
    if kind == "sptn3":
        I, J, K, L, M = (case[x] for x in "ijklm")
        nb, sel_u, sel_w = case["nb"], case["sel_u"], case["sel_w"]
        nnz_u, nnz_w = sel_u * (I // nb) * (J // nb) * (K // nb), sel_w * (K // nb) * (L // nb) * (M // nb)
        fibers = (1 - (1 - sel_u / nb ** 3) ** nb) * I * K           # (i,k) pairs that U stores
        rows_w = (1 - (1 - sel_w / nb ** 3) ** nb) * K * L
        # L multiply-adds per entry of U, and W's entries under k for every (i,k)
        return {"bytes": 12.0 * (nnz_u + fibers + I + nnz_w + rows_w + K) + 8.0 * (J * L + I * M),
                "flops": 2.0 * L * nnz_u + 2.0 * fibers * nnz_w / K}
    n_I, n_CP, n_E, squares, n_V = _lattice_sizes(case)
    if kind == "spchain3":
        # per stored (K,i): its u times their v, then its m times their v (a share of the block is stored)
        return {"bytes": 12.0 * (n_I + n_CP) + 12.0 * n_E, "flops": 2.0 * n_I * case["n_ao"] * KEEP_MO + 2.0 * n_E * case["n_ao"]}
    return {"bytes": 12.0 * n_E + 12.0 * n_V, "flops": 2.0 * squares}


def tolerance(case):
    if case["kind"] == "build":
        return "exact"
    # measured between kernels that sum in different orders: 2-norms off by up to 1.5e-15 of the result's, single
    # elements (differences of long sums over skewed slices) by up to 5.5e-13 of the root mean square
    return {"rel": 6e-15, "max": 2e-12}
