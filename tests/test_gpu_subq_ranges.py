"""Second pass of the sub-query update: lanes per run and counter copies follow the number of
bucket ranges and slabs; every target equals the oracle's on both sides of each rule."""
import numpy as np
import pytest

import oracle
import workloads as W
from tests.helpers import to_device_keys

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,d", [(2 ** 14, 2), (2 ** 14 + 1, 5), (2 ** 16, 4), (100003, 3), (2 ** 18, 6), (2 ** 20, 1)])
@pytest.mark.parametrize("n", [1, 2049, 30001])
def test_targets_equal_the_oracles(m, d, n):
    import paper_2402_15953_amd as csk
    graph, masks = W.chain(3), [0b01, 0b10, 0b11]
    rng = np.random.default_rng(n + d)
    rels = [rng.zipf(1.2, size=(n, len(graph.columns(k)))) % 2 ** 32 for k in range(graph.n_rel)]
    rels = [x.astype(np.uint32) for x in rels]
    info = oracle.analyze(graph)
    cs_, bn, js = oracle.draw_subq_coefficients(7, d, info.n_comp, len(info.edges))
    sq = csk.SubQueries(graph, masks, m, d, 7)
    for _ in range(2):   # the second call adds to counters that are not zero
        for k, keys in enumerate(rels):
            sq.update(k, to_device_keys(keys))
    _, target_of = sq.layout()
    for qi, mask in enumerate(masks):
        sub = oracle.subquery(graph, [e for e in range(32) if (mask >> e) & 1])
        for i, k in enumerate(sub.relations):
            ref = oracle.create_subq_sketch(info, sub.columns[i], rels[k], None, m, cs_, bn, js)
            assert np.array_equal(sq.read_target(int(target_of[qi, k])), 2 * ref), (mask, k)
    sq.close()
