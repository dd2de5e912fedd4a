"""Rows above the workgroup tables: chunk sums grouped by hash range, one workgroup per range.  Row lengths around the
chunk size and the lane groups that read a chunk's share (4, 8 and 16 chunks), more chunks than ranges, and ranges with
more clusters than the table, against the oracle, trace included.  The graphs are too large for the small-level route."""
from __future__ import annotations

import numpy as np
import pytest

import graphgen as gg
import oracle as O
from tests import gpu_util as U

pytestmark = pytest.mark.gpu
MOD, CPM = ((1, 1, True), O.VW_WEIGHTED_DEGREE), ((1, 50, False), O.VW_UNIT)


def _hubs(lengths, n, seed):
    rng = np.random.default_rng(seed)
    k = len(lengths)
    P = [np.stack([np.full(d, i), rng.choice(np.arange(k, n), size=d, replace=False)], axis=1) for i, d in enumerate(lengths)]
    P.append(rng.integers(k, n, size=(2 * n, 2)))
    P = np.concatenate(P)
    return gg.from_pairs(n, P, rng.integers(1, 9, size=len(P)), name="hubs")


@pytest.mark.parametrize("variant", [O.PLOUVAIN, O.PLEIDEN_PLUS])
@pytest.mark.parametrize("tuning", [{}, dict(bucket_max=[0] * 7), dict(bucket_max=[4, 8, 16, 32, 128, 128, 128])])
def test_hub_rows_around_the_chunks(variant, tuning):
    import paper_2608_01503_amd as L
    g = _hubs([2047, 2048, 2049, 4096, 8192, 8193, 16384, 16385, 32768, 32769, 60000], 90000, 3)
    ctx = U.ctx()
    old = ctx.get_tuning()
    ctx.set_tuning(L.lcc_default_tuning(**tuning))
    try:
        for lam, mode in (MOD, CPM):
            U.assert_parity(g, variant, lam, mode)
    finally:
        ctx.set_tuning(old)


@pytest.mark.parametrize("leaves", [2048 * 256, 2048 * 256 + 1, 1400000, 2048 * 1024 + 1])
def test_hub_of_more_chunks_than_ranges(leaves):
    """From singletons by labels, so that the first pass finds one cluster per leaf: 2048 * 1024
    + 1 leaves have 1,025 chunks, and two workgroups share each of 512 ranges."""
    g = gg.from_pairs(leaves + 1, np.stack([np.zeros(leaves, np.int64), np.arange(1, leaves + 1)], axis=1))
    init = np.random.default_rng(1).permutation(leaves + 1).astype(np.int32)
    for lam, mode in (MOD, CPM):
        U.assert_parity(g, O.LOUVAIN, lam, mode, opts_kw=dict(pass_limit=2), init=init)


def _fmix32(x):
    x = x.astype(np.uint64)
    for shift, mul in ((16, 0x85EBCA6B), (13, 0xC2B2AE35), (16, 1)):
        x = ((x ^ (x >> np.uint64(shift))) * np.uint64(mul)) & np.uint64(0xFFFFFFFF)
    return x


def test_hub_with_its_clusters_in_one_range():
    """A hub of 20 chunks whose 40,000 neighbours' labels all hash into one of the 20 ranges: the table of that range
    is split again until its parts fit."""
    n, d, chunks = 1 << 20, 40000, 20
    rng = np.random.default_rng(5)
    ranges = (_fmix32(np.arange(n)) * np.uint64(chunks)) >> np.uint64(32)
    labels = np.flatnonzero(ranges == 7)[:d]
    assert len(labels) == d
    rest = rng.permutation(np.setdiff1d(np.arange(n), labels))
    init = np.concatenate([rest[:1], labels, rest[1:]]).astype(np.int32)
    P = np.concatenate([np.stack([np.zeros(d, np.int64), np.arange(1, d + 1)], axis=1),
                        rng.integers(d + 1, n, size=(300000, 2))])
    g = gg.from_pairs(n, P, rng.integers(1, 9, size=len(P)))
    for lam, mode in (MOD, CPM):
        U.assert_parity(g, O.LOUVAIN, lam, mode, opts_kw=dict(pass_limit=2), init=init)
