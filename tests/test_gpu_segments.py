"""LDS-segmented update: the split into segments and tuple chunks follows the size of the
call, and a thread takes groups of tuples a block's stride apart; counters equal the
oracle's where a chunk, a group or a segment is partial, single or full."""
import numpy as np
import pytest
import torch

import workloads as W
from tests.helpers import oracle_sketches, to_device_keys

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,d,n", [(2, 9, 1), (2, 1, 70001), (1024, 5, 1023), (1024, 5, 4097), (1024, 5, 100000),
                                   (1000, 7, 8191), (16384, 5, 20479), (16384, 2, 65537), (16386, 3, 40000),
                                   (32768, 9, 40961), (65536, 9, 20001), (65534, 4, 12289)])
@pytest.mark.parametrize("weights", [None, "unit", "general"])
def test_balanced_segments(m, d, n, weights):
    import paper_2402_15953_amd as csk
    for graph in (W.chain(3), W.star(4)):
        rng = np.random.default_rng(m + d + n)
        rels = [rng.zipf(1.3, size=(n, len(graph.columns(k)))).astype(np.uint32) for k in range(graph.n_rel)]
        ws = None
        if weights:
            lim = 1 if weights == "unit" else 1 << 40
            ws = [np.where(rng.random(n) < 0.3, -1, 1) * rng.integers(1, lim + 1, n) for _ in rels]
        _, _, ref = oracle_sketches(graph, rels, ws, m, d, 11)
        sk = csk.Sketch(graph, m, d, 11)
        for k, keys in enumerate(rels):
            w = None if ws is None else torch.from_numpy(ws[k]).cuda()
            sk.update(k, to_device_keys(keys), w, strategy=csk.UPDATE_LDS_PRIVATE, unit_weights=weights == "unit")
        torch.cuda.synchronize()
        for k in range(graph.n_rel):
            assert np.array_equal(sk.read_sketch(k), ref[k]), (graph.name, k)
        sk.close()
