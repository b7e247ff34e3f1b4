"""GPU parity of the general trajectory scan's ranking floors: batches of two
or more query groups over stores of which each workgroup walks several
slices, so that later slices are ranked against a floor shared by the group's
workgroups.  Stores of many copies of a few maps (every kept match ties with
hundreds of others: the lowest indices must win) and stores with zero and NaN
maps, queries of either sign, for lists of 1, 4 and 8 in both types."""
import numpy as np
import pytest

import oracle
import synth
from parity import compare_topk, to_device

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("copies", [True, False])
@pytest.mark.parametrize("dtype,E,k,B,n", [("f32", 16, 4, 1000, 33001), ("f32", 8, 8, 600, 20011),
                                           ("f32", 60, 1, 600, 20003), ("bf16", 60, 8, 600, 20003),
                                           ("bf16", 16, 3, 600, 33007), ("f32", 60, 1, 600, 60003),
                                           ("bf16", 60, 8, 1000, 40003), ("bf16", 16, 3, 1000, 40007)])
def test_floors_keep_every_match(dtype, E, k, B, n, copies):
    import paper_2502_05370_amd as fm
    L = 5
    rng = np.random.default_rng(E + k + copies)
    maps = rng.dirichlet(np.ones(E), size=(40 if copies else n, L)).astype(np.float32)
    if copies:
        maps = maps[rng.integers(0, 40, n)]
    else:
        maps[7] = 0.0
        maps[8, 0, 0] = np.nan
        maps[n - 1, 0, E - 1] = np.nan
    q = maps[rng.integers(10, n - 1, B)].copy()
    q[1::2] += rng.normal(0, 0.05, size=q[1::2].shape).astype(np.float32)
    q[2::5] *= -1.0
    q[3] = 0.0
    depth = rng.integers(1, L + 1, B).astype(np.int32)
    if dtype == "bf16":
        maps, q = synth.bf16_bits(maps), synth.bf16_bits(q)
    store = fm.Store(n, L, E, 0, dtype)
    store.insert(to_device(maps, dtype))
    idx, score = (x.cpu().numpy() for x in fm.match_trajectory(store, to_device(q, dtype), to_device(depth, ""), k))
    rows = np.unique(np.concatenate([[0, 1, 2, 3, 4, B - 1], rng.integers(0, B, 18)]))
    oi, os_ = oracle.match_trajectory(maps, dtype, q[rows], depth[rows], k)

    def score_of(r, y):
        b = rows[r]
        return oracle.cosine(oracle.widen(q[b, :depth[b]], dtype), oracle.widen(maps[y, :depth[b]], dtype))

    rep = compare_topk(idx[rows], score[rows], oi, os_, score_of)
    assert not rep.failures, rep.failures[:3]
    if copies:   # copies score exactly alike: the k lowest indices of the best map, in order
        checked = 0
        for r, b in enumerate(rows):
            same = np.flatnonzero((maps[:, :depth[b]] == maps[idx[b, 0], :depth[b]]).all(axis=(1, 2)))
            if os_[r, -1] > os_[r, 0] - 1e-9 and b != 3:
                assert list(idx[b]) == list(same[:k]), (b, idx[b], same[:k])
                checked += 1
        assert checked > 5
