"""GPU parity of the scans that serve larger stores, on stores just large
enough for the dispatch to take them: the bf16 top-1 trajectory scan over its
layer geometries (several layers per k-step, one in one or two k-steps,
padding quads), the general trajectory scan with lists of 1, 4 and 8 in one
query group, and the top-1 semantic scan with one and two query groups.  The
oracle checks sampled queries against the whole store; zero and NaN maps,
scaled, zero and NaN queries are among them."""
import numpy as np
import pytest

import oracle
import synth
from parity import compare_topk, to_device

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,E,L,n,B,k", [("bf16", 8, 9, 40003, 300, 1), ("bf16", 16, 6, 40003, 300, 1),
                                             ("bf16", 20, 5, 40003, 257, 1), ("bf16", 32, 5, 40003, 300, 1),
                                             ("bf16", 64, 6, 40003, 600, 1), ("f32", 60, 6, 60001, 50, 1),
                                             ("f32", 16, 8, 70001, 20, 8), ("bf16", 60, 6, 60001, 90, 4),
                                             ("f32", 8, 12, 70001, 100, 4)])
def test_trajectory(dtype, E, L, n, B, k):
    import paper_2502_05370_amd as fm
    rng = np.random.default_rng(E + n + B)
    maps = rng.dirichlet(np.ones(E), size=(n, L)).astype(np.float32)
    q = maps[rng.integers(20, n, B)] + rng.uniform(0, 0.05, (B, L, E)).astype(np.float32)
    q[2] = 0.0
    q[3] *= -4.0
    q[4, 0, 0] = np.nan
    maps[10] = 0.0
    maps[11, 0, E - 1] = np.nan
    depth = rng.integers(1, L + 1, B).astype(np.int32)
    if dtype == "bf16":
        maps, q = synth.bf16_bits(maps), synth.bf16_bits(q)
    store = fm.Store(n, L, E, 0, dtype)
    store.insert(to_device(maps, dtype))
    idx, score = (x.cpu().numpy() for x in fm.match_trajectory(store, to_device(q, dtype), to_device(depth, ""), k))
    rows = np.unique(np.concatenate([np.arange(6), [B - 1], rng.integers(0, B, 14)]))
    oi, os_ = oracle.match_trajectory(maps, dtype, q[rows], depth[rows], k)

    def score_of(r, y):
        b = rows[r]
        return oracle.cosine(oracle.widen(q[b, :depth[b]], dtype), oracle.widen(maps[y, :depth[b]], dtype))

    rep = compare_topk(idx[rows], score[rows], oi, os_, score_of)
    assert not rep.failures, rep.failures[:3]
    assert list(idx[4]) == list(range(k)) and np.isnan(score[4]).all()


@pytest.mark.parametrize("n,d,B,k", [(60003, 256, 100, 1), (60003, 256, 300, 1), (120001, 128, 300, 8)])
def test_semantic(n, d, B, k):
    import paper_2502_05370_amd as fm
    rng = np.random.default_rng(n + B)
    e = rng.standard_normal((n, d)).astype(np.float32)
    q = e[rng.integers(20, n, B)] + 0.3 * rng.standard_normal((B, d)).astype(np.float32)
    q[0::5] *= -1.0
    q[1::5] *= 64.0
    q[3] = 0.0
    q[4, 7] = np.nan
    e[10] = 0.0
    e[11, 3] = np.nan
    e, q = synth.bf16_bits(e), synth.bf16_bits(q)
    store = fm.Store(n, 1, 4, d, "f32")
    store.insert(to_device(np.full((n, 1, 4), 0.25, np.float32), "f32"), to_device(e, "bf16"))
    idx, score = (x.cpu().numpy() for x in fm.match_semantic(store, to_device(q, "bf16"), k))
    rows = np.unique(np.concatenate([np.arange(6), [B - 1], rng.integers(0, B, 14)]))
    oi, os_ = oracle.match_semantic(e, q[rows], k)
    e64, q64 = oracle.widen(e, "bf16"), oracle.widen(q, "bf16")
    rep = compare_topk(idx[rows], score[rows], oi, os_, lambda r, y: oracle.cosine(q64[rows[r]], e64[y]))
    assert not rep.failures, rep.failures[:3]
    assert list(idx[4]) == list(range(k)) and np.isnan(score[4]).all()
