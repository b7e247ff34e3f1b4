"""GPU parity of the split-k semantic scan at the edges of its five shapes:
16-query tiles, steps of 1 or 4 blocks of 16 maps, k-steps that do not divide
evenly over the wavefronts (d = 128: four k-steps for eight), one match and the
dense form, with zero, scaled, infinite and NaN queries and zero and NaN stored
embeddings, against the CPU oracle on the same arrays; and lists of 4 and 8 of
the same inputs, which k_sem_scan serves.  Index and score rules
as for every match (parity.compare_topk)."""
import numpy as np
import pytest

import oracle
import synth
from parity import SCORE_TOL, compare_topk, to_device

pytestmark = pytest.mark.gpu


def _embeddings(rng, n, d):
    x = rng.standard_normal((8, d))[rng.integers(0, 8, n)] + 0.3 * rng.standard_normal((n, d))
    return (x / np.linalg.norm(x, axis=1, keepdims=True)).astype(np.float32)


@pytest.mark.parametrize("n,d,B", [(1, 128, 1), (15, 128, 5), (17, 384, 16), (250, 4096, 17), (1003, 1152, 33),
                                   (1003, 256, 65), (4100, 2048, 8), (4100, 640, 129), (333, 1024, 300),
                                   (9001, 1024, 70), (1052, 4096, 450), (12007, 2048, 100)])
def test_split_scan_matches_oracle(n, d, B):
    import paper_2502_05370_amd as fm
    rng = np.random.default_rng(n + d + B)
    e, q = _embeddings(rng, n, d), _embeddings(rng, B, d)
    q[0::3] *= 64.0
    q[1::3] *= -1.0 / 64.0
    if B > 4:
        q[2] = 0.0
        q[3, 5] = np.nan
        q[4, d - 1] = np.inf
    if n > 12:
        e[10] = 0.0
        e[11, 3] = np.nan
    e, q = synth.bf16_bits(e), synth.bf16_bits(q)
    maps = rng.dirichlet(np.ones(4), size=(n, 2)).astype(np.float32)
    store = fm.Store(n, 2, 4, d, "f32")
    store.insert(to_device(maps, "f32"), to_device(e, "bf16"))
    e64, q64 = oracle.widen(e, "bf16"), oracle.widen(q, "bf16")
    finite = [b for b in range(B) if np.isfinite(q64[b]).all()]
    lb, le = np.zeros(B, np.int32), np.full(B, 2, np.int32)
    for k in (1, 3, 8):
        idx, score = (x.cpu().numpy() for x in fm.match_semantic(store, to_device(q, "bf16"), k))
        fi, fs, mask, _ = (x.cpu().numpy() for x in fm.match_semantic_select(
            store, to_device(q, "bf16"), to_device(lb, ""), to_device(le, ""), k=k, tau=0.7))
        assert np.array_equal(fi, idx) and np.array_equal(fs, score, equal_nan=True)
        oi, os_ = oracle.match_semantic(e, q[finite], k)
        rep = compare_topk(idx[finite], score[finite], oi, os_, lambda r, y: oracle.cosine(q64[finite[r]], e64[y]))
        assert not rep.failures, (k, rep.failures[:3])
        om, _ = oracle.select_prefetch(maps, "f32", idx, score, lb, le, 0, float(np.float32(0.7)), 1, 4, 0)
        assert np.array_equal(mask.view(np.uint64), om)
        # a query with a NaN or an infinity: every cosine is NaN, the lowest indices win
        m = min(k, n)
        for b in set(range(B)) - set(finite):
            assert list(idx[b, :m]) == list(range(m)) and np.isnan(score[b, :m]).all()
            assert (idx[b, m:] == -1).all()
    # the dense form: every cosine
    dense = fm.debug_scores(store, q_sem=to_device(q, "bf16")).cpu().numpy()
    for b in finite[:40]:
        ref = oracle.semantic_scores(e64, q64[b])
        assert np.array_equal(np.isnan(ref), np.isnan(dense[b]))
        assert np.nanmax(np.abs(dense[b] - ref)) <= SCORE_TOL
