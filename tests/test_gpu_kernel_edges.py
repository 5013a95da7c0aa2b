"""GPU tests at the sizes where a kernel's split of the work has its edges:
wave and tile boundaries, remainders, the switch from one variant to another.
Integer results must be equal; float64 sums carry a derived bound."""
import numpy as np
import pytest
import torch

import paper_2511_06600_amd as hef
from synth.hypergraph import Hypergraph
from tests.gpu_common import say, to_device

pytestmark = pytest.mark.gpu


def _hg(n, sizes, seed, w=None):
    """Hyperedges of the given sizes over random distinct nodes."""
    rng = np.random.default_rng(seed)
    pins = [np.sort(rng.choice(n, size=s, replace=False)) for s in sizes]
    eptr = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    m = len(sizes)
    w = np.ones(m, np.float32) if w is None else w
    return Hypergraph(n=n, m=m, eptr=eptr, pins=np.concatenate(pins).astype(np.int32), w=w)


def _mixed_sizes(m, seed, long_at=()):
    s = np.random.default_rng(seed).integers(2, 7, m)
    for i, k in long_at:
        s[i] = k
    return [int(x) for x in s]


@pytest.mark.parametrize("m", [1, 63, 64, 65, 200])
def test_device_validation_at_wave_edges(m):
    """A wave validates 64 hyperedges: a repeated, descending or out-of-range
    pin is found at the first and last pin of the wave's first, last and a
    long hyperedge, a bad weight anywhere; equal pins in neighbouring
    hyperedges are no fault."""
    say(f"case: device validation m={m}")
    n = 500
    h = _hg(n, _mixed_sizes(m, m, [(m // 2, 300)]), 7 * m)
    label = torch.zeros(n, dtype=torch.int32, device="cuda")

    def status(pins, w=h.w):
        dh = hef.DeviceHypergraph.from_arrays(n, m, h.eptr, pins, w)
        try:
            hef.conductance(dh, label, 1)
        except hef.HefError as e:
            return str(e)
        return ""

    assert status(h.pins) == ""
    for e in {0, m // 2, m - 1, min(m - 1, 63), min(m - 1, 64)}:
        a, b = int(h.eptr[e]), int(h.eptr[e + 1])
        for j, v in ((a + 1, h.pins[a]), (b - 1, h.pins[b - 2]), (b - 1, n), (a, -1)):
            p = h.pins.copy()
            p[j] = v
            assert "code 4" in status(p), (e, j, v)
        w = h.w.copy()
        w[e] = 0.0
        assert "code 8" in status(h.pins, w)
    # the last pin of a hyperedge may equal the first of the next
    if m > 1:
        p = h.pins.copy()
        e = m // 2 - 1
        a, b, c = (int(h.eptr[i]) for i in (e, e + 1, e + 2))
        if p[b - 2] < p[b]:
            p[b - 1] = p[b]
        assert status(p) == ""


def _star_of(n, bound, seed, pool=None, parts=3):
    """Hyperedges around node 0 whose other pins are `bound` distinct nodes,
    then two small ones that repeat some of them."""
    rng = np.random.default_rng(seed)
    others = rng.permutation(np.arange(1, n) if pool is None else pool)[:bound]
    edges = [np.concatenate([[0], c]) for c in np.array_split(others, min(parts, bound))]
    edges += [np.array([0, others[0]]), np.array([1, 2, 3])]
    edges = [np.sort(e) for e in edges]
    eptr = np.concatenate([[0], np.cumsum([len(e) for e in edges])]).astype(np.int64)
    w = rng.uniform(0.5, 2.0, len(edges)).astype(np.float32)
    return Hypergraph(n=n, m=len(edges), eptr=eptr, pins=np.concatenate(edges).astype(np.int32),
                      w=w)


@pytest.mark.parametrize("bound", [62, 63, 64, 510, 511, 512, 2047, 2049, 4500, "one class"])
def test_rating_class_edges(bound):
    """The node's table changes at 64 and 512 triples and is swept in hash
    classes above 2048 neighbours; in the last case the neighbours all fall
    in one of the first sweep's four classes, which overflows its table."""
    from oracle import rating as orat
    say(f"case: rating bound={bound}")
    n, pool = 6000, None
    if bound == "one class":
        n = 60000
        q = np.arange(4, n, dtype=np.uint64)
        h = (q * 2654435769) & 0xFFFFFFFF
        pool = q[((h >> 18) & 3) == 1].astype(np.int64)[:4500]
        bound = len(pool)
    hg = _star_of(n, bound, 11, pool)
    R = np.random.default_rng(5).uniform(0.01, 1.0, hg.m).astype(np.float32)
    best, val = hef.rating(to_device(hg), torch.as_tensor(R, device="cuda"), 0.0)
    nodes = np.unique(np.concatenate([[0, 1, 2, 3], hg.pins[:200:17], [n - 1]]))
    rb, rv = orat.best_neighbours(hg.n, hg.m, hg.eptr, hg.pins, hg.w, R, 0.0, nodes)
    assert np.array_equal(best.cpu().numpy()[nodes], rb)
    assert np.array_equal(val.cpu().numpy()[nodes], rv)
