"""GPU parity of the row kernels (selection, misses, priority order) at the
edges of their row widths: 8, 16, 32 or 64 lanes hold a row's experts, so E on
and beside each width, with a layer count that leaves the last wavefront of
a query partly filled.  Rows hold many equal values, zeros of both signs, NaN
and infinities.  Everything is exact: both sides rank the same stored
values and sum them in float64 in rank order."""
import numpy as np
import pytest

import oracle
import synth
from parity import to_device

pytestmark = pytest.mark.gpu


def _maps(rng, n, L, E, dtype):
    maps = (np.round(rng.dirichlet(np.ones(E), size=(n, L)) * 32) / 32).astype(np.float32)   # many ties
    maps[0] = 0.25
    maps[1, 0] = -0.0
    maps[1, 0, E // 2] = 0.0
    maps[2, 0, E - 1] = np.nan
    maps[2, 1, 0] = np.inf
    maps[3] = rng.dirichlet(np.ones(E), size=L)
    return synth.bf16_bits(maps) if dtype == "bf16" else maps


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("E", [1, 4, 7, 8, 9, 16, 17, 32, 33, 60, 64])
def test_rows_match_oracle(E, dtype):
    import paper_2502_05370_amd as fm
    L, n, B, k = 7, 24, 13, 3
    rng = np.random.default_rng(E)
    maps = _maps(rng, n, L, E, dtype)
    store = fm.Store(n, L, E, 0, dtype)
    store.insert(to_device(maps, dtype))
    idx = np.stack([rng.permutation(n)[:k] for _ in range(B)]).astype(np.int32)
    idx[:4, 0] = np.arange(4)
    idx[4] = -1
    idx[5, 1:] = -1
    score = np.sort(rng.uniform(-0.2, 1.0, size=(B, k)).astype(np.float32), axis=1)[:, ::-1].copy()
    score[6] = -0.5               # no positive weight: the plain mean
    score[7, 0] = np.nan          # most conservative threshold, weight 0
    lb = rng.integers(-1, 3, size=B).astype(np.int32)
    le = rng.integers(L - 2, L + 2, size=B).astype(np.int32)
    lb[8], le[8] = 5, 5           # an empty range
    t = lambda x: to_device(x, "")  # noqa: E731
    for blend in (0, 1):
        for mode, tau, k_min, k_max in ((0, 0.6, 0, E), (0, 0.6, 0, min(E, 3)), (0, 0.0, 0, E), (1, 0.0, min(E, 2), E),
                                        (0, 2.0, 0, 0)):
            mask, count = fm.select_prefetch(store, t(idx), t(score), t(lb), t(le), tau=tau, k_min=k_min, k_max=k_max,
                                             mode=mode, blend=blend)
            om, oc = oracle.select_prefetch(maps, dtype, idx, score, lb, le, mode, float(np.float32(tau)), k_min, k_max,
                                            blend)
            assert np.array_equal(mask.cpu().numpy().view(np.uint64), om), (blend, mode, tau, k_max)
            assert np.array_equal(count.cpu().numpy(), oc), (blend, mode, tau, k_max)
            l_now = rng.integers(-1, L, size=B).astype(np.int32)
            order, pri, nc = fm.priority_order(store, t(idx), t(score), mask, l_now=t(l_now), blend=blend)
            oo, op, on = oracle.priority_order(maps, dtype, idx, score, blend, oracle.PRI_PREFETCH, om, l_now=l_now)
            gp = pri.cpu().numpy()
            assert np.array_equal(nc.cpu().numpy(), on) and np.array_equal(order.cpu().numpy(), oo)
            assert ((gp == op) | (np.isnan(gp) & np.isnan(op))).all()
            # misses of the sets, the queries being stored maps
            q = maps[np.maximum(idx[:, 0], 0)]
            for K in {1, max(1, E // 2), E}:
                miss = fm.miss_count(store, to_device(q, dtype), mask, K, t(lb), t(le))
                assert np.array_equal(miss.cpu().numpy(), oracle.miss_counts(q, dtype, om, K, lb, le)), K
