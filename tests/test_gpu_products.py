"""Modular products summed as the last transform pass makes their factors: every length from
one pass to two, conjugated relations, the general plan's sum by Parseval, and sub-queries
that need more primes than the call before; integers equal the oracle's."""
import numpy as np
import pytest
import torch

import oracle
import workloads as W
from tests.helpers import oracle_sketches, to_device_keys

pytestmark = pytest.mark.gpu


def _relations(graph, n, seed, weight):
    rng = np.random.default_rng(seed)
    rels = [rng.zipf(1.3, size=(n, len(graph.columns(k)))).astype(np.uint32) for k in range(graph.n_rel)]
    return rels, [rng.integers(1, weight + 1, n) for _ in rels]


@pytest.mark.parametrize("graph", [W.chain(3), W.chain(4), W.chain(5), W.star(4), W.fig3_query()], ids=lambda g: g.name)
@pytest.mark.parametrize("m,d", [(2, 1), (64, 5), (1024, 4), (2048, 1), (4096, 5), (8192, 5), (16384, 2), (32768, 1),
                                 (1000, 3), (2047, 1), (2049, 5), (5000, 2), (16385, 1)])
def test_products_of_every_length(graph, m, d):
    import paper_2402_15953_amd as csk
    rels, ws = _relations(graph, 3000, m + d, 1 << 24)
    info, _, ref = oracle_sketches(graph, rels, ws, m, d, 13)
    reps, _ = oracle.estimate(info, ref, m, method="ntt")
    sk = csk.Sketch(graph, m, d, 13)
    for k, keys in enumerate(rels):
        sk.update(k, to_device_keys(keys), torch.from_numpy(ws[k]).cuda())
    for _ in range(2):   # the second call computes as many primes as the first one needed
        got = sk.estimate(reps=True)
        if all(abs(x) < 2 ** 125 for x in reps):
            assert got["rep_ints"] == reps
    sk.close()


@pytest.mark.parametrize("m,d", [(64, 5), (1024, 3), (4096, 1), (8192, 5), (32768, 2)])
def test_more_primes_than_the_call_before(m, d):
    import paper_2402_15953_amd as csk
    graph = W.chain(4)
    subs = W.connected_subqueries(graph)
    small, ws_small = _relations(graph, 50, 1, 1)
    big, ws_big = _relations(graph, 3000, 2, 1 << 28)
    sq = csk.SubQueries(graph, subs, m, d, 5)
    fresh = csk.SubQueries(graph, subs, m, d, 5)
    for k in range(graph.n_rel):
        for target in (sq, fresh):
            target.update(k, to_device_keys(small[k]), torch.from_numpy(ws_small[k]).cuda())
    sq.estimate_all()
    sq.estimate_all()    # no primes needed: the next call computes none beforehand
    for k in range(graph.n_rel):
        for target in (sq, fresh):
            target.update(k, to_device_keys(big[k]), torch.from_numpy(ws_big[k]).cuda())
    want = [fresh.estimate(q) for q in range(len(subs))]
    got = sq.estimate_all()
    assert [e["value"] for e in got] == [e["value"] for e in want]
    assert [e["exact"] for e in got] == [e["exact"] for e in want]
    assert any(e["n_modular"] for e in got)
    sq.close()
    fresh.close()
