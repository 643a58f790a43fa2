"""Small calls: a workgroup per repetition for updates of few tuples, tables and results of
small estimates passed through pinned memory without copies; both sides of each limit."""
import numpy as np
import pytest

import workloads as W
from tests.helpers import oracle_sketches, to_device_keys

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [64, 1000])
@pytest.mark.parametrize("d,n", [(1, 1), (5, 257), (5, 13056), (5, 13057), (9, 7168), (9, 7169)])
def test_global_update_split_over_repetitions(m, d, n):
    import paper_2402_15953_amd as csk
    graph = W.chain(3)
    rng = np.random.default_rng(n + d)
    rels = [rng.zipf(1.3, size=(n, len(graph.columns(k)))).astype(np.uint32) for k in range(graph.n_rel)]
    _, _, ref = oracle_sketches(graph, rels, None, m, d, 3)
    sk = csk.Sketch(graph, m, d, 3)
    for k, keys in enumerate(rels):
        sk.update(k, to_device_keys(keys), strategy=csk.UPDATE_GLOBAL_ATOMIC)
        assert np.array_equal(sk.read_sketch(k), ref[k]), k
    sk.close()


@pytest.mark.parametrize("d", [4, 5])
@pytest.mark.parametrize("nq", [1, 30, 102, 103, 128, 129, 300])
def test_estimates_on_both_sides_of_the_copies(d, nq):
    import paper_2402_15953_amd as csk
    rng = np.random.default_rng(d)
    plain = []
    for graph, m, weight in ((W.chain(3), 256, 1), (W.chain(2), 64, 1), (W.star(4), 128, 1 << 40)):
        sk = csk.Sketch(graph, m, d, 7)
        for k in range(graph.n_rel):
            keys = rng.zipf(1.2, size=(500, len(graph.columns(k)))).astype(np.uint32)
            sk.update(k, to_device_keys(keys), None if weight == 1 else to_device_weights(weight, 500))
        plain.append(sk)
    alone = [sk.estimate(reps=True) for sk in plain]
    b = csk.Batch()
    for _ in range(2):
        got = b.estimate([plain[q % 3] for q in range(nq)], reps=True)
        assert got == [alone[q % 3] for q in range(nq)]
    b.close()
    for sk in plain:
        sk.close()


def to_device_weights(weight, n):
    import torch
    return torch.full((n,), weight, dtype=torch.int64, device="cuda")
