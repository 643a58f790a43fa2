"""Second pass of the partition update: lanes per run and counter copies follow the number of
bucket ranges and repetitions; counters equal the oracle's on both sides of each rule."""
import numpy as np
import pytest

import workloads as W
from tests.helpers import oracle_sketches, to_device_keys

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,d", [(2 ** 16 + 2, 5), (2 ** 17, 3), (2 ** 18, 2), (10 ** 6, 4), (10 ** 6, 5),
                                 (2 ** 20, 4), (2 ** 20, 5)])
@pytest.mark.parametrize("n", [1, 4097, 70001])
def test_counter_copies_and_run_widths(m, d, n):
    import paper_2402_15953_amd as csk
    graph = W.chain(3)
    rng = np.random.default_rng(n + d)
    rels = [(rng.zipf(1.2, size=(n, len(graph.columns(k)))) % 2 ** 32).astype(np.uint32) for k in range(graph.n_rel)]
    _, _, ref = oracle_sketches(graph, rels, None, m, d, 9)
    sk = csk.Sketch(graph, m, d, 9)
    for _ in range(2):   # the second call adds to counters that are not zero
        for k, keys in enumerate(rels):
            sk.update(k, to_device_keys(keys), strategy=csk.UPDATE_PARTITION)
    for k in range(graph.n_rel):
        assert np.array_equal(sk.read_sketch(k), 2 * ref[k]), k
    sk.close()
