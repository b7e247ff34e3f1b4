"""GPU parity of the split-depth trajectory scan at the edges of its shapes:
16-query tiles in groups of one, two and four, steps of one and two blocks of
16 maps, fewer k-steps than wavefronts and numbers that do not divide evenly,
several layers per k-step (E = 4, 8, 16), one in one or two (E = 20, 60, 64),
stores of one map to several steps per workgroup, all depths from 1 to L, a
zero and a negated query, zero and NaN maps, lists of 1, 4 and 8, both types;
and the match-and-select form against the match followed by the selection."""
import numpy as np
import pytest

import oracle
import synth
from parity import compare_topk, to_device

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("E,L,n,B", [(8, 32, 1, 1), (8, 5, 15, 5), (16, 3, 17, 16), (20, 7, 250, 17), (60, 24, 1003, 33),
                                     (64, 9, 333, 65), (8, 32, 4100, 100), (60, 6, 4100, 200), (4, 10, 2050, 9),
                                     (16, 32, 9001, 40)])
def test_split_depth_matches_oracle(E, L, n, B, dtype):
    import paper_2502_05370_amd as fm
    rng = np.random.default_rng(E * L + n + B)
    maps = rng.dirichlet(np.ones(E), size=(n, L)).astype(np.float32)
    q = maps[rng.integers(0, n, B)] + rng.uniform(0, 0.05, (B, L, E)).astype(np.float32)
    if B > 4:
        q[2] = 0.0
        q[3] *= -1.0
    if n > 12:
        maps[10] = 0.0
        maps[11, 0, E - 1] = np.nan
    depth = rng.integers(1, L + 1, B).astype(np.int32)
    depth[0] = L
    depth[B // 2] = 1
    if dtype == "bf16":
        maps, q = synth.bf16_bits(maps), synth.bf16_bits(q)
    store = fm.Store(n, L, E, 0, dtype)
    store.insert(to_device(maps, dtype))
    rows = np.unique(np.concatenate([np.arange(min(B, 6)), [B // 2, B - 1], rng.integers(0, B, 20)]))
    qt, dt = to_device(q, dtype), to_device(depth, "")
    lb, le = to_device(np.zeros(B, np.int32), ""), to_device(np.full(B, L, np.int32), "")
    q64, m64 = oracle.widen(q, dtype), oracle.widen(maps, dtype)
    for k in (1, 3, 8):
        idx, score = (x.cpu().numpy() for x in fm.match_trajectory(store, qt, dt, k))
        oi, os_ = oracle.match_trajectory(maps, dtype, q[rows], depth[rows], k)

        def score_of(r, y):
            b = rows[r]
            return oracle.cosine(q64[b, :depth[b]], m64[y, :depth[b]])

        rep = compare_topk(idx[rows], score[rows], oi, os_, score_of)
        assert not rep.failures, (k, rep.failures[:3])
        fi, fs, mask, count = fm.match_trajectory_select(store, qt, dt, lb, le, k=k, tau=0.7, k_max=min(E, 8))
        assert np.array_equal(fi.cpu().numpy(), idx) and np.array_equal(fs.cpu().numpy(), score, equal_nan=True)
        m2, c2 = fm.select_prefetch(store, fi, fs, lb, le, tau=0.7, k_max=min(E, 8))
        assert bool((m2 == mask).all()) and bool((c2 == count).all())
    assert store.check() == 0


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("E,L,n,B", [(8, 32, 700, 200), (16, 9, 4100, 100), (60, 7, 3001, 200),
                                     (20, 11, 4100, 100), (60, 7, 9001, 100)])
def test_deep_non_finite_values_stay_out_of_shallower_tiles(E, L, n, B, dtype):
    """A NaN or an infinity stored in the last layer ranks its map last for the
    queries that reach that layer.  A 16-query tile (of the depth-sorted batch)
    whose deepest query ends before that layer group keeps its finite scores,
    whatever deeper tiles share its workgroup."""
    import paper_2502_05370_amd as fm
    for k in (1, 4):
        assert fm.debug_scan_name(L, E, n, B, k, dtype).startswith("k_traj_split 2")
    rng = np.random.default_rng(E + n)
    maps = rng.dirichlet(np.ones(E), size=(n, L)).astype(np.float32)
    lpg = 32 // E if E >= 8 and 32 % E == 0 else 1
    shallow = (L - 1) // lpg * lpg   # the layers before the last layer's group
    depth = np.full(B, L, np.int32)
    depth[16:] = rng.integers(1, shallow + 1, B - 16)   # one tile of deep queries, then shallow tiles
    q = maps[rng.integers(0, n, B)] + rng.uniform(0, 0.02, (B, L, E)).astype(np.float32)
    src = rng.integers(20, n, B)
    q[16:] = maps[src[16:]]          # shallow queries copy the maps that hold the values
    maps[src[16::2], L - 1, 0] = np.nan
    maps[src[17::2], L - 1, E - 1] = np.inf
    order = rng.permutation(B)
    q, depth = np.ascontiguousarray(q[order]), np.ascontiguousarray(depth[order])
    if dtype == "bf16":
        maps, q = synth.bf16_bits(maps), synth.bf16_bits(q)
    store = fm.Store(n, L, E, 0, dtype)
    store.insert(to_device(maps, dtype))
    q64, m64 = oracle.widen(q, dtype), oracle.widen(maps, dtype)
    for k in (1, 4):
        idx, score = (x.cpu().numpy() for x in fm.match_trajectory(store, to_device(q, dtype), to_device(depth, ""), k))
        with np.errstate(invalid="ignore"):
            oi, os_ = oracle.match_trajectory(maps, dtype, q, depth, k)
            rep = compare_topk(idx, score, oi, os_, lambda r, y: oracle.cosine(q64[r, :depth[r]], m64[y, :depth[r]]))
        assert not rep.failures, (k, len(rep.failures), rep.failures[:3])
        assert np.isfinite(score).all()
