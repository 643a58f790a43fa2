"""Sub-queries of one base query share relation sketches, which one call transforms once:
every sub-query's estimate equals the one computed alone, whichever plans the sharing
sub-queries take and however their repetitions pair up."""
import numpy as np
import pytest

import workloads as W
from tests.helpers import to_device_keys

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("graph", [W.chain(5), W.star(4), W.fig3_query()], ids=lambda g: g.name)
@pytest.mark.parametrize("d", [1, 4, 5])
@pytest.mark.parametrize("m", [256, 1000, 8192])
def test_shared_transforms(graph, m, d):
    import paper_2402_15953_amd as csk
    subs = W.connected_subqueries(graph)
    subs += subs[:2]   # a sub-query asked for twice
    sq = csk.SubQueries(graph, subs, m, d, 5)
    rng = np.random.default_rng(m + d)
    for k in range(graph.n_rel):
        keys = rng.zipf(1.2, size=(30000, len(graph.columns(k)))).astype(np.uint32)
        sq.update(k, to_device_keys(keys))
    alone = [sq.estimate(q) for q in range(len(subs))]
    for _ in range(2):   # the second call computes as many primes as the first one needed
        together = sq.estimate_all()
        assert [e["value"] for e in together] == [e["value"] for e in alone]
        assert all(e["exact"] for e in together)
    sq.close()
