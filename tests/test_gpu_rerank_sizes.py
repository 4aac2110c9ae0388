"""fp32 re-rank at the sizes where its paths meet: rows that end inside a group of loads, lists that end inside a pass of
rows, ranks counted (up to 128 candidates) and sorted, repeated and absent candidates, fewer candidates than results.
Against binary64 sums in numpy.  Needs a real MI355X."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("metric", ["l2sq", "ip"])
@pytest.mark.parametrize("d", [1, 7, 24, 25, 32, 33, 100, 257])
@pytest.mark.parametrize("kc,k", [(1, 1), (5, 9), (32, 10), (33, 33), (100, 10), (129, 40), (256, 300), (257, 20), (700, 700)])
def test_rerank(metric, d, kc, k):
    from paper_2110_08919_amd import lpq
    g = np.random.default_rng(1000 * d + kc)
    n, nq = 900, 6
    x, q = g.integers(-8, 9, size=(n, d)).astype(np.float32), g.integers(-8, 9, size=(nq, d)).astype(np.float32)
    cand = g.integers(-3, n + 3, size=(nq, kc)).astype(np.int32)
    cand[:, kc // 2] = cand[:, 0]                                 # the same row twice
    ids, dists = lpq.rerank_f32(torch.as_tensor(x).cuda(), torch.as_tensor(q).cuda(), torch.as_tensor(cand).cuda(), k, metric)
    ids, dists = ids.cpu().numpy(), dists.cpu().numpy()
    for i in range(nq):
        live = [c for c in cand[i] if 0 <= c < n]
        v = [float(((x[c] - q[i]).astype(np.float64) ** 2).sum()) if metric == "l2sq" else -float((x[c].astype(np.float64) * q[i]).sum())
             for c in live]
        order = sorted(range(len(live)), key=lambda j: (v[j], live[j]))[:k]
        none = k - len(order)
        assert ids[i].tolist() == [int(live[j]) for j in order] + [-1] * none
        want = [v[j] if metric == "l2sq" else -v[j] for j in order] + [np.inf if metric == "l2sq" else -np.inf] * none
        assert dists[i].tolist() == [float(np.float32(w)) for w in want]


# no two distances alike: ranks by the upper halves of the keys; absent candidates agree in them and take the sort
@pytest.mark.parametrize("absent", [0, 3])
@pytest.mark.parametrize("d,kc,k", [(17, 1, 1), (16, 100, 10), (17, 64, 70), (40, 33, 5), (129, 128, 128), (64, 127, 20), (33, 129, 129)])
def test_rerank_of_distinct_candidates(d, kc, k, absent):
    from paper_2110_08919_amd import lpq
    g = np.random.default_rng(d + kc)
    x, q = g.standard_normal((900, d)).astype(np.float32), g.standard_normal((50, d)).astype(np.float32)
    cand = np.stack([g.permutation(900)[:kc] for _ in range(50)]).astype(np.int32)
    cand[:, kc - min(absent, kc):] = -1
    ids, dists = (t.cpu().numpy() for t in lpq.rerank_f32(*(torch.as_tensor(a).cuda() for a in (x, q, cand)), k, "l2sq"))
    for i in range(50):
        live = cand[i][cand[i] >= 0]
        v = ((x[live].astype(np.float64) - q[i]) ** 2).sum(1)
        order = np.argsort(v)[:k]
        assert ids[i].tolist() == live[order].tolist() + [-1] * (k - len(order))
        assert np.allclose(dists[i][:len(order)], v[order], rtol=1e-6) and np.all(np.isinf(dists[i][len(order):]))
