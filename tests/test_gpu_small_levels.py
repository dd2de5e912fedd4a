"""Small levels run in one launch of a team of workgroups; with kernel timing on, the same calls take the per-bucket
launches.  Labels, exact objective, levels, flags and the whole trace must be the same on both routes: every row
length around the edges of the team's row kernels, the smallest graphs, and entry counts around the size limit."""
from __future__ import annotations

import numpy as np
import pytest

import graphgen as gg
import oracle as O
from tests import gpu_util as U

pytestmark = pytest.mark.gpu
MOD, CPM = ((1, 1, True), O.VW_WEIGHTED_DEGREE), ((1, 20, False), O.VW_UNIT)


def _rows(lengths, n, seed):
    """A graph with one row of each given length (more or less) over sparse random edges."""
    rng = np.random.default_rng(seed)
    pairs = [np.stack([np.full(d, i), rng.choice(np.arange(len(lengths), n), size=d, replace=False)], axis=1)
             for i, d in enumerate(lengths)]
    pairs.append(rng.integers(0, n, size=(2 * n, 2)))
    P = np.concatenate(pairs)
    return gg.from_pairs(n, P, rng.integers(1, 50, size=len(P)), name="rows")


GRAPHS = {
    "rows": lambda: _rows([3, 4, 5, 8, 9, 16, 17, 31, 32, 33, 63, 64, 65, 127, 128, 129, 511, 512, 513, 1024, 1025], 3000, 1),
    "long rows": lambda: _rows([4096, 4097, 8191, 8192, 8193, 9500], 40000, 2),
    "pair": lambda: gg.from_pairs(2, [(0, 1)]),
    "star": lambda: gg.from_pairs(1026, [(0, i) for i in range(1, 1026)]),
    "limit": lambda: gg.random_gnp(2200, 0.1075, 3, w_max=3),  # about 2^19 entries
    "above limit": lambda: gg.random_gnp(2200, 0.1095, 3, w_max=3),
}


@pytest.mark.parametrize("name", GRAPHS)
@pytest.mark.parametrize("variant", [O.PLOUVAIN, O.PLEIDEN, O.PLEIDEN_PLUS, O.LOUVAIN])
def test_team_equals_bucket_launches(name, variant):
    import torch
    import paper_2608_01503_amd as L
    g = GRAPHS[name]()
    buckets = L.Context(0)
    buckets.profile_enable(["single"])
    team = L.Context(0)
    opts = [{}, dict(pass_limit=3), dict(symmetry=2, phases=((0, 1, 6),)), dict(pass_limit=0)]
    for (lam, mode), kw in [(MOD, opts[0]), (CPM, opts[0]), (CPM, opts[1]), (MOD, opts[2]), (MOD, opts[3])]:
        dev = U.device_graph(g, mode)
        got = [c.cluster(dev, lam, variant, L.lcc_default_options(**kw), trace_capacity=1 << 14) for c in (buckets, team)]
        (la, a), (lb, b) = got
        assert np.array_equal(la.cpu().numpy(), lb.cpu().numpy()), (name, lam, kw)
        assert (a.N, a.num_clusters, a.levels, a.flags) == (b.N, b.num_clusters, b.levels, b.flags)
        assert np.array_equal(a.trace, b.trace)
    buckets.close()
    team.close()


# next levels with rows around the lane groups, the bitmap and the dense table of the contraction, and refinement trees
# around a lane group, a wavefront and the LDS sort
NEXT = {
    "stars": lambda: gg.from_pairs(6000, [(c, 1000 * c + i) for c, d in enumerate([15, 16, 17, 63, 64, 65]) for i in range(1, 3 * d)]
                                   + [(i, i + 1000) for i in range(200, 5000, 7)]),
    "wide star": lambda: gg.from_pairs(40001, [(0, i) for i in range(1, 40001)]),
    "dense rows": lambda: _rows([900, 1020, 1024, 1028, 1100, 2050], 9000, 4),
    "many vertices": lambda: gg.lattice(220, 220, 0.05, 100, 3),
}


@pytest.mark.parametrize("name", NEXT)
@pytest.mark.parametrize("variant", [O.PLEIDEN, O.PLEIDEN_PLUS, O.PLOUVAIN])
def test_team_next_level_equals_launches(name, variant):
    import torch
    import paper_2608_01503_amd as L
    g = NEXT[name]()
    buckets = L.Context(0)
    buckets.profile_enable(["single"])
    team = L.Context(0)
    rng = np.random.default_rng(3)
    init = rng.integers(0, g.n // 40, g.n).astype(np.int32)
    # without passes the alternate move decides: from three clusters its events fill a workgroup's sort and more
    few = rng.integers(0, 3, g.n).astype(np.int32)
    for lam, mode, lab, opt in [(*MOD, None, {}), (*CPM, None, {}), ((0, 1, False), O.VW_UNIT, None, {}), (*CPM, init, {}),
                                (*CPM, init, dict(pass_limit=0)), (*CPM, few, dict(pass_limit=0)), (*MOD, few, dict(pass_limit=0))]:
        dev = U.device_graph(g, mode)
        kw = {} if lab is None else dict(init=torch.from_numpy(lab).cuda())
        got = [c.cluster(dev, lam, variant, L.lcc_default_options(seed=5, **opt), trace_capacity=1 << 14, **kw) for c in (buckets, team)]
        (la, a), (lb, b) = got
        assert np.array_equal(la.cpu().numpy(), lb.cpu().numpy()), (name, lam)
        assert (a.N, a.num_clusters, a.levels, a.flags) == (b.N, b.num_clusters, b.levels, b.flags)
        assert np.array_equal(a.trace, b.trace)
    buckets.close()
    team.close()


@pytest.mark.parametrize("name", ["rows", "limit"])
def test_team_constrained_equals_launches(name):
    import torch
    import paper_2608_01503_amd as L
    g = GRAPHS[name]()
    buckets = L.Context(0)
    buckets.profile_enable(["single"])
    team = L.Context(0)
    B = torch.from_numpy(np.random.default_rng(4).integers(0, 30, g.n).astype(np.int32)).cuda()
    dev = U.device_graph(g, CPM[1])
    (la, a), (lb, b) = [c.cluster(dev, CPM[0], O.PLOUVAIN, L.lcc_default_options(), trace_capacity=1 << 14, constraint=B) for c in (buckets, team)]
    assert np.array_equal(la.cpu().numpy(), lb.cpu().numpy()) and (a.N, a.levels, a.flags) == (b.N, b.levels, b.flags)
    assert np.array_equal(a.trace, b.trace)
    buckets.close()
    team.close()


def _set(a, i, v):
    a[i] = v


# (what, change of offsets, indices and weights): the smallest input for every check of the setup
FAULTS = [
    ("none", lambda o, i, w: None),
    ("descending offsets", lambda o, i, w: _set(o, 5, o[6] + 1)),
    ("first offset", lambda o, i, w: _set(o, 0, 1)),
    ("last offset", lambda o, i, w: _set(o, -1, o[-1] + 2)),
    ("index n", lambda o, i, w: _set(i, 9, len(o) - 1)),
    ("index -1", lambda o, i, w: _set(i, 0, -1)),
    ("self loop", lambda o, i, w: _set(i, o[3], 3)),
    ("unsorted", lambda o, i, w: _set(i, slice(o[4], o[4] + 2), i[o[4]:o[4] + 2][::-1].copy())),
    ("zero weight", lambda o, i, w: _set(w, 3, 0)),
    ("one-sided weight", lambda o, i, w: _set(w, 3, w[3] + 1)),
]


@pytest.mark.parametrize("what,change", FAULTS, ids=[f[0] for f in FAULTS])
@pytest.mark.parametrize("offsets32", [False, True])
def test_team_setup_equals_launches(what, change, offsets32):
    import torch
    import paper_2608_01503_amd as L
    g = gg.random_gnp(300, 0.03, 100, w_max=5)
    off, idx, w = g.off.copy(), g.idx.copy(), g.w.copy()
    change(off, idx, w)
    h = gg.Graph(n=g.n, off=off, idx=idx, w=w)
    buckets = L.Context(0)
    buckets.profile_enable(["single"])
    team = L.Context(0)
    for lam, mode, kw in [(*MOD, {}), (*CPM, {}), (*CPM, dict(validate=0)), ((1, 3, False), O.VW_UNIT, dict(no_w=True))]:
        kw = dict(kw)
        with_w = not kw.pop("no_w", False)
        if "validate" in kw and what not in ("none", "index n", "index -1", "first offset"):
            continue  # without the checks only structural faults are the library's to find
        dev = U.device_graph(h, mode, offsets32=offsets32, with_w=with_w)
        got = []
        for c in (buckets, team):
            for init in (None, torch.full((g.n,), g.n, dtype=torch.int32, device="cuda:0")):
                try:
                    lab, r = c.cluster(dev, lam, O.PLOUVAIN, L.lcc_default_options(**kw), init=init)
                    got.append((lab.cpu().numpy().tolist(), r.N, r.num_clusters, r.levels, r.flags))
                except L.LccError as e:
                    got.append(str(e))
        assert got[:2] == got[2:], (what, lam, kw)
    buckets.close()
    team.close()


@pytest.mark.parametrize("n", [1023, 1024, 1025, 1088, 2047, 2048, 2049, 5000])
def test_alternate_move_by_radix_sort_equals_team(n):
    """Four records per mover around the sort's tiles of 4096: from one cluster each by label, nearly every vertex moves."""
    import torch
    import paper_2608_01503_amd as L
    g = gg.random_gnp(n, 8.0 / n, 7, w_max=4)
    buckets = L.Context(0)
    buckets.profile_enable(["single"])
    team = L.Context(0)
    init = torch.from_numpy(np.random.default_rng(2).permutation(n).astype(np.int32)).cuda()
    dev = U.device_graph(g, CPM[1])
    (la, a), (lb, b) = [c.cluster(dev, CPM[0], O.PLEIDEN, L.lcc_default_options(pass_limit=0), trace_capacity=1 << 14, init=init)
                        for c in (buckets, team)]
    assert np.array_equal(la.cpu().numpy(), lb.cpu().numpy()) and (a.N, a.levels, a.flags) == (b.N, b.levels, b.flags)
    assert np.array_equal(a.trace, b.trace) and (a.trace[:, 0] == 3).any()
    buckets.close()
    team.close()
