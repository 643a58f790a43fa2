"""The one-join update kernels take a tuple's bucket and sign from the leading bits of
rotated polynomials, and fall back to the exact residue where those bits are too near a
rounding limit.  The arithmetic is modelled here in Python integers (CPU), with
coefficients placed so that residues land on and next to every limit; on the GPU, keys whose
hashes fall nearest the limits are compared with the oracle through each kernel."""
import random

import numpy as np
import pytest
import torch

import oracle
import workloads as W
from tests.helpers import oracle_sketches, to_device_keys

P = (1 << 61) - 1
M32, M64 = (1 << 32) - 1, (1 << 64) - 1


def _rotr(a, k):
    return a * pow(2, -k, P) % P


def _hstep(v, x, a):
    lo = (v & M32) * x
    t = (v >> 32) * x + (lo >> 32)
    assert t <= M64
    return (((t & 0x1FFFFFFF) << 32) | (lo & M32)) + (t >> 29) + a


def _hstep_wrap(v, x, a):
    assert v < 1 << 63
    lo = (v & M32) * x
    t = (v >> 32) * x + (lo >> 32)
    return ((((t & M32) << 32) | (lo & M32)) + 8 * (t >> 32) + a) & M64


def _bin_fast(b0, b1, x, k):
    """(bucket, whether the exact hash is asked for) from the leading bits."""
    q = b1 >> 58
    B = 8 * b1 + q + (((8 * b1) & P) + q >= P)
    assert B == b1 * (1 << 64) // P
    t = ((x * (B & M32) >> 32) + x * (B >> 32)) & M32
    r = (t << k) + (b0 >> (29 - k))
    assert r <= M64
    return (r >> 32) & ((1 << k) - 1), (r & M32) >= (1 << 32) - 2 * (1 << k) - 2


def _neg_fast(a, x):
    v = _hstep_wrap(_hstep(a[3], x, a[2]), x, a[1])
    t = (((v & M32) * x >> 32) + (v >> 32) * x + (a[0] >> 32)) & M32
    return (t >> 28) & 1, ((t << 4) & M32) >= (1 << 32) - 16 * 24


@pytest.mark.parametrize("k", [1, 2, 10, 16, 18, 20])
def test_leading_bits_agree_with_the_residue_or_ask_for_it(k):
    rng = random.Random(k)
    asked = 0
    for i in range(20000):
        x = rng.choice([0, 1, M32, M32 - 1, 1 << 31, rng.getrandbits(32), rng.getrandbits(8)])
        b1 = rng.choice([0, 1, P - 1, rng.randrange(P), rng.randrange(P)])
        # the divided residue at, or next to, a multiple of p / 2^k (in steps up to 2^40)
        near = (rng.randrange(1 << k) << (61 - k)) + rng.choice([-1, 1, 0]) * rng.randrange(1 << rng.randrange(1, 41))
        b0 = (near - b1 * x) % P
        h = (b0 + b1 * x) % P * (1 << k) % P
        j, again = _bin_fast(b0, b1, x, k)
        assert again or j == h % (1 << k)
        a = [0] + [rng.choice([0, P - 1, rng.randrange(P)]) for _ in range(3)]
        near = (rng.randrange(2) << 60) + rng.choice([-1, 1, 0]) * rng.randrange(1 << rng.randrange(1, 45))
        a[0] = (near - sum(a[e] * x ** e for e in (1, 2, 3))) % P
        s = sum(c * x ** e for e, c in enumerate(a)) % P * 2 % P & 1
        g, sagain = _neg_fast(a, x)
        assert sagain or g == s
        asked += again + sagain
    assert asked > 100   # the limits were reached


@pytest.mark.parametrize("k", [1, 11, 16, 20])
def test_random_hashes_agree(k):
    rng = random.Random(100 + k)
    for _ in range(20000):
        x = rng.getrandbits(32)
        c = [rng.randrange(P) for _ in range(6)]
        j, again = _bin_fast(_rotr(c[0], k), _rotr(c[1], k), x, k)
        assert again or j == (c[0] + c[1] * x) % P % (1 << k)
        g, sagain = _neg_fast([_rotr(v, 1) for v in c[2:]], x)
        assert not sagain and g == (c[2] + c[3] * x + c[4] * x * x + c[5] * x ** 3) % P & 1


@pytest.mark.gpu
@pytest.mark.parametrize("m,strategy", [(2, 2), (1 << 10, 2), (1 << 16, 2), (1 << 17, 2), (1 << 18, 4), (1 << 20, 4)])
@pytest.mark.parametrize("r", [2, 3, 5])
def test_keys_next_to_the_limits(m, strategy, r):
    """strategy 2: LDS segments, 4: partition; chains of two- and one-column relations, and
    (r = 5) a star's centre of four columns."""
    import paper_2402_15953_amd as csk
    graph = W.star(5) if r == 5 else W.chain(r)
    if r == 5 and strategy == 4:
        strategy = 2
    d, seed = 3, 4242
    info = oracle.analyze(graph)
    co = oracle.draw_coefficients(seed, d, len(info.edges), info.n_comp)
    b = co.bin_array()
    x = np.random.default_rng(3).integers(0, 1 << 32, size=1 << 15, dtype=np.uint64)
    xs = [int(v) for v in x]
    k = m.bit_length() - 1
    pick = []
    for t in range(d):
        for q in range(info.n_comp):
            b0, b1 = _rotr(int(b[t, q, 0]), k), _rotr(int(b[t, q, 1]), k)
            dist = np.array([(b0 + b1 * v) % P % (1 << (61 - k)) for v in xs], dtype=np.float64)
            order = np.argsort(dist)
            pick += [order[:200], order[-200:]]   # just above and just below a limit
    keys = x[np.concatenate(pick)].astype(np.uint32)
    rng = np.random.default_rng(4)
    n = len(keys)
    rels = [np.stack([rng.permutation(keys) for _ in graph.columns(c)], axis=1) for c in range(graph.n_rel)]
    _, _, ref = oracle_sketches(graph, rels, None, m, d, seed)
    sk = csk.Sketch(graph, m, d, seed)
    for c, kk in enumerate(rels):
        sk.update(c, to_device_keys(kk), strategy=strategy)
    torch.cuda.synchronize()
    for c in range(graph.n_rel):
        assert np.array_equal(sk.read_sketch(c), ref[c]), (n, c)
    sk.close()
