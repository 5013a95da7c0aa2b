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


@pytest.mark.parametrize("bound", [62, 63, 64, 510, 511, 512, 3071, 3073, 4500, "one class"])
def test_rating_class_edges(bound):
    """The node's table changes at 64 and 512 triples and is swept in hash
    classes above 3072 neighbours; in the last case the neighbours all fall
    in one class of the first two sweeps, which overflows its table."""
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


@pytest.mark.parametrize("nnz", [2, 1023, 1025, 4096, 4097, 8192, 8193, 16385, 70001, 1048577])
def test_sort_and_compaction_sizes(nnz):
    """The incidence sort runs in one workgroup up to 8192 items (4 or 8 a
    thread), in tiles of 1024 up to 2^20 and of 4096 above; node counts
    that need one digit pass or two, of 8 bits and of 9.  The operator's rows depend on every
    node's hyperedges being complete and in order."""
    say(f"case: sort sizes nnz={nnz}")
    for n in (200, 60000, 70000):
        if nnz == 2 and n != 200:
            continue
        m = max(nnz // 3, 1)
        rng = np.random.default_rng(nnz + n)
        first = rng.integers(0, n - 2 * (nnz - 2 * m + 1), m) if n > 2 * (nnz - 2 * m + 1) \
            else rng.integers(0, n - 3, m)
        sizes = np.full(m, 2)
        left = nnz - 2 * m
        sizes[rng.permutation(m)[:left]] += 1 if left <= m else 0
        eptr = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
        pins = (np.repeat(first, sizes) + np.arange(eptr[-1]) - np.repeat(eptr[:-1], sizes))
        h = Hypergraph(n=n, m=m, eptr=eptr, pins=pins.astype(np.int32), w=np.ones(m, np.float32))
        label = torch.arange(n, dtype=torch.int32, device="cuda")
        # every node its own cluster: vol = degree, cut = degree (all split)
        cut, vol, _, _ = hef.conductance(to_device(h), label, n)
        deg = np.bincount(h.pins, minlength=n).astype(np.float64)
        assert np.array_equal(vol.cpu().numpy(), deg) and np.array_equal(cut.cpu().numpy(), deg)
        # star operator on hyperedge indicators: y_u = s_u sum_e alpha_e x_e
        x = torch.zeros((n + m, 1), device="cuda")
        x[n:, 0] = torch.arange(m, device="cuda") % 13
        y = hef.debug_apply(to_device(h), 0, x).cpu().numpy()[:n, 0].astype(np.float64)
        inv = 1.0 / sizes
        db = np.bincount(h.pins, weights=np.repeat(inv, sizes), minlength=n)
        ref = np.bincount(h.pins, weights=np.repeat(inv * (np.arange(m) % 13), sizes), minlength=n)
        ref = np.where(db > 0, ref / np.sqrt(np.where(db > 0, db, 1.0)), 0.0)
        # float32 scales and terms: (degree + 4) roundings of relative 2^-24
        tol = (deg.max() + 4) * 2.0 ** -24
        assert np.abs(y - ref).max() <= tol * max(np.abs(ref).max(), 1.0)


@pytest.mark.parametrize("k,b,basis", [(4, 1, "fp32"), (5, 2, "bf16"), (17, 8, "fp32"),
                                       (9, 4, "fp64")])
@pytest.mark.parametrize("nodes", ["many", "few"])
def test_long_hyperedge_ratios(k, b, basis, nodes):
    """Hyperedges of 32, 33, 64, 65 and 700 pins, first and last among them,
    side by side; with few nodes per pin only longer ones go to the separate
    pass.  Q_H and R of the returned pool against float64 on that pool: the
    maxima are exact, a float64 sum of m terms is within m 2^-53 of any other
    order, R carries one float32 rounding of the numerator and one of the
    ratio."""
    from oracle import resistance as orr
    say(f"case: long hyperedges k={k} b={b} {basis} {nodes}")
    n = 3000 if nodes == "many" else 710
    sizes = [700, 33, 32, 65, 64] + _mixed_sizes(900, 3) + [40, 300, 33]
    sizes += [] if nodes == "many" else [60] * 300
    h = _hg(n, sizes, 9, np.random.default_rng(1).uniform(0.5, 2, len(sizes)).astype(np.float32))
    R, qh, chi = hef.resistance(to_device(h), hef.Params(k=k, b=b, basis=basis), return_pool=True)
    c = chi.cpu().double().numpy()
    s = orr.edge_spread(h.eptr, h.pins, c)
    q = h.w.astype(np.float64) @ s
    qg = qh.cpu().numpy()
    assert np.abs(qg - q).max() <= 2 * h.m * 2.0 ** -53 * q.max()
    ref = (s / q[None, :]).max(1)
    np.testing.assert_allclose(R.cpu().numpy(), ref, rtol=2.0 ** -22, atol=0)


@pytest.mark.parametrize("b", [1, 2, 4, 8])
@pytest.mark.parametrize("n,m", [(127, 255), (128, 256), (129, 257), (300, 20)])
def test_krylov_step_at_workgroup_edges(b, n, m):
    """The Lanczos apply takes 128 node rows of both expansions or 256
    hyperedge rows per workgroup and hands the next product its gather rows:
    the estimate against the oracle at the edges of both, and against the
    single-expansion passes' columns (which keep the separate prep pass)."""
    from oracle import resistance as orr
    from tests.gpu_common import r_errors, starts
    k = 3
    say(f"case: krylov step n={n} m={m} b={b}")
    h = _hg(n, _mixed_sizes(m, n + m), n)
    Xs, Xc, xs, xc = starts(h, b)
    est = orr.resistance(h.n, h.m, h.eptr, h.pins, h.w, Xs, Xc, k)
    R, qh, _ = hef.resistance(to_device(h), hef.Params(k=k, b=b), xs, xc)
    norm, p999, _ = r_errors(R.cpu().numpy(), est.R)
    assert norm <= 1e-4 and p999 <= 1e-4
    star = hef.resistance(to_device(h), hef.Params(k=k, b=b, star_only=True), xs, None,
                          return_pool=True)[2] if b * k > 4 else None
    both = hef.resistance(to_device(h), hef.Params(k=k, b=b), xs, xc, return_pool=True)[2]
    # the star columns come first in the joint Gram-Schmidt
    if star is not None:
        d = (both[:, :k * b] - star).abs().max().item()
        assert d <= 1e-6


@pytest.mark.parametrize("k,b", [(5, 1), (20, 2), (6, 4), (17, 4), (17, 8), (5, 16)])
def test_gradient_with_long_hyperedges(k, b):
    """Hyperedges of 32, 33, 64 and 300 pins (a workgroup each above 32) in the
    score adjoint, narrow and wide lane groups, every block width, pools of one
    to three 128-column blocks, against the float64 autograd
    oracle at the adjoint tests' bound of 1e-3."""
    from oracle import gradient as ogr
    from tests.gpu_common import starts
    say(f"case: adjoint long hyperedges k={k} b={b}")
    sizes = [300, 32, 33, 64] + _mixed_sizes(700, 3) + [65, 33]
    w = np.random.default_rng(2).uniform(0.5, 2.0, len(sizes)).astype(np.float32)
    h = _hg(800, sizes, 21, w)
    Xs, Xc, xs, xc = starts(h, b)
    coef = np.random.default_rng(3).standard_normal(h.m).astype(np.float32)
    _, ref, _ = ogr.loss_and_grad(h.n, h.m, h.eptr, h.pins, h.w, Xs, Xc, k, coef)
    dw = hef.resistance_backward(to_device(h), hef.Params(k=k, b=b),
                                 torch.as_tensor(coef, device="cuda"), xs, xc).cpu().numpy()
    assert np.linalg.norm(dw - ref) <= 1e-3 * np.linalg.norm(ref)


@pytest.mark.parametrize("n", [1, 2, 63, 1024, 16383, 16384, 16385, 40000])
def test_level_maps_at_scan_sizes(n):
    """Labels, clusters and pairs are placed by scans that run in one workgroup
    up to 16384 items: one clustering level against the oracle, bit for bit."""
    from oracle import clustering as ocl
    if n < 4:
        h = _hg(4, [2] * n, 3)
    else:
        h = _hg(n, _mixed_sizes(max(n // 2, 1), n), n)
    say(f"case: level map n={h.n} m={h.m}")
    rng = np.random.default_rng(n)
    K = 8
    p = hef.Params(k=4, b=1)
    R = rng.random(h.m).astype(np.float32)
    chi = rng.standard_normal((h.n, K)).astype(np.float32) / np.sqrt(h.n)
    qh = rng.uniform(0.5, 2.0, K)
    cl, nc, eta = hef.cluster_level(to_device(h), p, torch.as_tensor(R, device="cuda"), None,
                                    torch.as_tensor(chi.astype(np.float32), device="cuda"),
                                    torch.as_tensor(qh, device="cuda"))
    chi32 = chi.astype(np.float32)
    ref = ocl.cluster_level(h.n, h.m, h.eptr, h.pins, R, np.zeros(h.n, np.float32), chi32, qh,
                            0.5, True)
    assert nc == ref.n_clusters
    assert np.array_equal(cl.cpu().numpy(), ref.label)
    assert np.array_equal(eta.cpu().numpy(), ref.eta.astype(np.float32))


@pytest.mark.parametrize("size", [32, 33, 64, 65, 256, 257, 700])
def test_level_and_rebuild_with_long_segments(size):
    """Segments around the lengths at which a wave takes over: the level (its
    Eq. (15) sums run in pin order), the attach chains of the union-find and
    the coarse hypergraph against the oracle, bit for bit."""
    from oracle import clustering as ocl
    say(f"case: long segments size={size}")
    n = 1500
    sizes = [size, 3, size + 1] + _mixed_sizes(1200, size) + [size]
    h = _hg(n, sizes, size)
    # a hub in `size` hyperedges more
    rng = np.random.default_rng(size)
    extra = np.stack([np.zeros(size, np.int64), 1 + rng.choice(n - 1, size, replace=False)], 1)
    eptr = np.concatenate([h.eptr, h.eptr[-1] + 2 * np.arange(1, size + 1)])
    pins = np.concatenate([h.pins, extra.reshape(-1)]).astype(np.int32)
    m = len(eptr) - 1
    h = Hypergraph(n=n, m=m, eptr=eptr, pins=pins, w=np.ones(m, np.float32))
    K = 8
    R = rng.random(m).astype(np.float32)
    eta = (0.05 * rng.random(n)).astype(np.float32)
    chi = (0.1 * rng.standard_normal((n, K))).astype(np.float32)
    qh = rng.random(K) + 0.5
    dh = to_device(h)
    cl, nc, eo = hef.cluster_level(dh, hef.Params(k=4, b=1), torch.as_tensor(R, device="cuda"),
                                   torch.as_tensor(eta, device="cuda"),
                                   torch.as_tensor(chi, device="cuda"),
                                   torch.as_tensor(qh, device="cuda"))
    ref = ocl.cluster_level(n, m, h.eptr, h.pins, R, eta, chi, qh, 0.5, True)
    assert nc == ref.n_clusters and np.array_equal(cl.cpu().numpy(), ref.label)
    assert np.array_equal(eo.cpu().numpy().view(np.uint32), ref.eta.view(np.uint32))
    out, kept = hef.rebuild(dh, cl, nc)
    m2, ep, pn, w2, kp = ocl.rebuild(m, h.eptr, h.pins, h.w, ref.label)
    assert out.m == m2 and np.array_equal(out.eptr.cpu().numpy(), ep)
    assert np.array_equal(out.pins.cpu().numpy(), pn) and np.array_equal(kept.cpu().numpy(), kp)


@pytest.mark.parametrize("m", [1, 63, 64, 65, 200])
def test_conductance_at_wave_edges(m):
    """A wave takes 64 hyperedges' pins, 256 positions at once: hyperedges of
    one cluster but for one pin, at either end or across a chunk's edge, and
    whole ones.  Unit weights: the sums are whole numbers and must be equal."""
    say(f"case: conductance wave edges m={m}")
    n = 900
    for long in (2, 62, 64, 255, 256, 257, 700):
        h = _hg(n, _mixed_sizes(m, m + long, [(0, long), (m - 1, long), (m // 2, long)]), m + long)
        deg = np.bincount(h.pins, minlength=n)
        a, b = int(h.eptr[m // 2]), int(h.eptr[m // 2 + 1])
        for j in (a, a + min(63, long - 1), a + min(64, long - 1), b - 1, -1):
            label = np.zeros(n, np.int32)
            if j >= 0:
                label[h.pins[j]] = 2
            cut, vol, phi, _ = hef.conductance(to_device(h), torch.as_tensor(label, device="cuda"), 3)
            inside = np.add.reduceat(label[h.pins] == 0, h.eptr[:-1])
            k = int(((inside > 0) & (inside < np.diff(h.eptr))).sum())
            two = int((inside < np.diff(h.eptr)).sum())
            assert two == k  # no hyperedge lies in the single node's cluster
            assert cut.cpu().tolist() == [k, 0, k]
            assert vol.cpu().tolist() == [deg[label == 0].sum(), 0, deg[label == 2].sum()]


@pytest.mark.parametrize("k,b,m", [(3, 1, 127), (7, 1, 128), (5, 2, 129), (8, 4, 40), (17, 8, 300),
                                   (4, 2, 65536), (4, 2, 65537), (10, 4, 65409),
                                   (17, 8, 32768), (17, 8, 32769)])
def test_quadratic_forms_at_block_edges(k, b, m):
    """Q_H is summed over blocks of 128 hyperedges, up to 512 of them (256 of
    more than 256 columns) with four times the threads: blocks full and one hyperedge long, lane groups of 2 to
    64 lanes, either side of the rule.  Bounds as in
    test_long_hyperedge_ratios."""
    from oracle import resistance as orr
    say(f"case: quadratic forms k={k} b={b} m={m}")
    n = 2000
    rng = np.random.default_rng(m + k)
    sizes = rng.integers(2, 5, m)
    eptr = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    first = np.repeat(rng.integers(0, n - 40, m), sizes)
    pins = first + 11 * (np.arange(eptr[-1]) - np.repeat(eptr[:-1], sizes))
    w = rng.uniform(0.5, 2, m).astype(np.float32)
    h = Hypergraph(n=n, m=m, eptr=eptr, pins=pins.astype(np.int32), w=w)
    R, qh, chi = hef.resistance(to_device(h), hef.Params(k=k, b=b), return_pool=True)
    s = orr.edge_spread(h.eptr, h.pins, chi.cpu().double().numpy())
    q = w.astype(np.float64) @ s
    assert np.abs(qh.cpu().numpy() - q).max() <= 2 * max(m, 2) * 2.0 ** -53 * q.max()
    ok = q > 0
    ref = (s[:, ok] / q[ok]).max(1)
    np.testing.assert_allclose(R.cpu().numpy(), ref, rtol=2.0 ** -22, atol=0)


NARROW = [(1, 1, "star"), (1, 1, "both"), (3, 1, "clique"), (2, 1, "both"), (1, 2, "both"),
          (1, 4, "star")]  # pools of 1, 2, 3, 4, 4 and 4 columns


@pytest.mark.parametrize("basis", ["fp32", "bf16", "fp64"])
@pytest.mark.parametrize("m", [127, 128, 129, 70000])
def test_narrow_pools_are_scored(m, basis):
    """Pools of at most four columns, one lane's worth: every hyperedge is
    scored, up to and above the 512 blocks of the variant for few hyperedges
    and with long ones among them, in the checked call and in the unchecked
    one.  Bounds as in test_long_hyperedge_ratios."""
    from oracle import resistance as orr
    n = 900
    rng = np.random.default_rng(m)
    sizes = rng.integers(2, 5, m)
    if m > 100:
        sizes[[0, m // 2, m - 1]] = [33, 300, 64]
    step = np.where(sizes > 4, 1, 11)
    eptr = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    first = rng.integers(0, n - (sizes - 1) * step)
    pins = np.repeat(first, sizes) + np.repeat(step, sizes) * (
        np.arange(eptr[-1]) - np.repeat(eptr[:-1], sizes))
    w = rng.uniform(0.5, 2, m).astype(np.float32)
    h = Hypergraph(n=n, m=m, eptr=eptr, pins=pins.astype(np.int32), w=w)
    dh = to_device(h)
    for k, b, pool in NARROW:
        say(f"case: narrow pool k={k} b={b} {pool} m={m} {basis}")
        kw = dict(k=k, b=b, basis=basis, star_only=pool == "star", clique_only=pool == "clique")
        R, qh, chi = hef.resistance(dh, hef.Params(**kw), return_pool=True)
        s = orr.edge_spread(h.eptr, h.pins, chi.cpu().double().numpy())
        q = w.astype(np.float64) @ s
        assert np.abs(qh.cpu().numpy() - q).max() <= 2 * max(m, 2) * 2.0 ** -53 * q.max()
        ok = q > 0
        ref = (s[:, ok] / q[ok]).max(1)
        np.testing.assert_allclose(R.cpu().numpy(), ref, rtol=2.0 ** -22, atol=0)
        Ru, qu, cu = hef.resistance_static(dh, hef.Params(assume_valid=True, **kw),
                                           return_pool=True)
        assert torch.equal(Ru, R) and torch.equal(qu, qh) and torch.equal(cu, chi)


@pytest.mark.parametrize("k,b", [(1, 1), (2, 1), (1, 2)])
def test_narrow_pools_in_gradient_and_coarsening(k, b):
    """Pools of two and four columns through the adjoint (against the float64
    autograd oracle, at the adjoint tests' bound of 1e-3) and through two
    levels of coarsening, level 1 from the library's own resistances against
    the oracle bit for bit."""
    from oracle import clustering as ocl
    from oracle import gradient as ogr
    from tests.gpu_common import starts
    say(f"case: narrow pools, gradient and coarsening k={k} b={b}")
    sizes = _mixed_sizes(700, 3) + [65, 33, 32]
    w = np.random.default_rng(2).uniform(0.5, 2.0, len(sizes)).astype(np.float32)
    h = _hg(800, sizes, 21, w)
    dh = to_device(h)
    Xs, Xc, xs, xc = starts(h, b)
    coef = np.random.default_rng(3).standard_normal(h.m).astype(np.float32)
    _, ref, Rr = ogr.loss_and_grad(h.n, h.m, h.eptr, h.pins, h.w, Xs, Xc, k, coef)
    dR = torch.as_tensor(coef, device="cuda")
    dw = hef.resistance_backward(dh, hef.Params(k=k, b=b), dR, xs, xc)
    assert np.linalg.norm(dw.cpu().numpy() - ref) <= 1e-3 * np.linalg.norm(ref)
    R, tape = hef.resistance_taped(dh, hef.Params(k=k, b=b), xs, xc)
    assert torch.equal(hef.resistance_backward(dh, hef.Params(k=k, b=b), dR, xs, xc, tape=tape), dw)
    assert np.linalg.norm(R.cpu().numpy() - Rr) <= 1e-4 * np.linalg.norm(Rr)
    p = hef.Params(k=k, b=b, levels=2)
    cl, nc, R0, _, lev = hef.coarsen_levels(dh, p)
    R1, qh, chi = hef.resistance(dh, hef.Params(k=k, b=b), return_pool=True)
    assert torch.equal(R0, R1) and torch.equal(lev[0]["R"], R1) and torch.equal(lev[0]["qh"], qh)
    out = ocl.cluster_level(h.n, h.m, h.eptr, h.pins, R1.cpu().numpy(), np.zeros(h.n, np.float32),
                            chi.cpu().numpy(), qh.cpu().numpy(), 0.5, True)
    assert np.array_equal(lev[0]["label"].cpu().numpy(), out.label)
    assert np.array_equal(lev[0]["eta"].cpu().numpy().view(np.uint32), out.eta.view(np.uint32))
    assert len(lev) == 2 and (lev[1]["R"] > 0).any() and (lev[1]["qh"] > 0).any()


@pytest.mark.parametrize("at", ["first", "middle", "two"])
def test_rebuild_with_a_giant_hyperedge_before_others(at):
    """A hyperedge of more than 16384 pins (left to the global sort) with
    hyperedges after it: the emission that runs before the host learns of it
    places those by its count.  The coarse hypergraph and the level counts of
    a coarsening against the oracle."""
    from oracle import clustering as ocl
    n = 20000
    giant = {"first": [0], "middle": [1500], "two": [3, 2000]}[at]
    sizes = _mixed_sizes(3000, 5, [(i, 17000 + i) for i in giant])
    h = _hg(n, sizes, 31)
    say(f"case: giant hyperedge {at} n={n} m={h.m} nnz={h.eptr[-1]}")
    dh = to_device(h)
    rng = np.random.default_rng(8)
    nc = 5000
    label = np.concatenate([np.arange(nc), rng.integers(0, nc, n - nc)]).astype(np.int32)
    out, kept = hef.rebuild(dh, torch.as_tensor(label, device="cuda"), nc)
    m2, ep, pn, w2, kp = ocl.rebuild(h.m, h.eptr, h.pins, h.w, label)
    assert out.m == m2 and np.array_equal(out.eptr.cpu().numpy(), ep)
    assert np.array_equal(out.pins.cpu().numpy(), pn) and np.array_equal(kept.cpu().numpy(), kp)
    assert np.array_equal(out.w.cpu().numpy(), w2)
    *_, lev = hef.coarsen_levels(dh, hef.Params(k=4, b=1, levels=2))
    m1, e1, *_ = ocl.rebuild(h.m, h.eptr, h.pins, h.w, lev[0]["label"].cpu().numpy())
    assert (lev[1]["m"], lev[1]["nnz"]) == (m1, int(e1[-1]))


@pytest.mark.parametrize("K", [4, 8, 300])
@pytest.mark.parametrize("tiny", ["one", "most", "all"])
def test_best_neighbour_with_tiny_quadratic_forms(K, tiny):
    """Quadratic forms below 2.9e-39, whose reciprocal float32 cannot hold, and
    either side of that: the float16 screen decides nothing there and every
    candidate gets its exact distance.  Nodes with one candidate and with more
    than the 64 survivors kept at once, entries of both signs and zeros; the
    level against the oracle, bit for bit."""
    from oracle import clustering as ocl
    n = 700
    say(f"case: tiny quadratic forms K={K} {tiny}")
    h = _hg(n, _mixed_sizes(350, K, [(0, 150), (200, 90)]), K)
    rng = np.random.default_rng(K)
    chi = (1e-3 * rng.choice([-1.0, 1.0, 0.0, 0.5], (n, K))
           * (1 + 1e-2 * rng.random((n, K)))).astype(np.float32)
    qh = rng.uniform(0.5, 2.0, K)
    some = {"one": slice(0, 1), "most": slice(0, K - 1), "all": slice(0, K)}[tiny]
    qh[some] = rng.choice([1e-40, 2e-39, 2.9e-39, 3e-39, 1e-38], K)[some]
    qh[0] = 1e-40
    R = rng.random(h.m).astype(np.float32)
    out = hef.cluster_level(to_device(h), hef.Params(k=K // 4, b=2), torch.as_tensor(R, device="cuda"),
                            None, torch.as_tensor(chi, device="cuda"),
                            torch.as_tensor(qh, device="cuda"))
    ref = ocl.cluster_level(n, h.m, h.eptr, h.pins, R, None, chi, qh, 0.5, True)
    assert out[1] == ref.n_clusters and np.array_equal(out[0].cpu().numpy(), ref.label)
    assert np.array_equal(out[2].cpu().numpy().view(np.uint32), ref.eta.view(np.uint32))


def test_level_sorts_fit_just_above_a_million_pins():
    """Slightly more than 2^20 pins and about as many clusters as nodes: the
    level's largest sort is not its pins' but its clusters', in the smaller
    tiles.  The level against the oracle, bit for bit (no local clustering),
    and a coarsening whose level scratch is the largest part."""
    from oracle import clustering as ocl
    n, m, nnz = 1_000_000, 500_000, 1_100_000
    say(f"case: level sorts n={n} m={m} nnz={nnz}")
    rng = np.random.default_rng(4)
    sizes = np.full(m, 2)
    sizes[rng.permutation(m)[:nnz - 2 * m]] += 1
    eptr = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    assert eptr[-1] == nnz
    pins = np.repeat(rng.integers(0, n - 30, m), sizes) + 13 * (
        np.arange(nnz) - np.repeat(eptr[:-1], sizes))
    w = rng.uniform(0.5, 2.0, m).astype(np.float32)
    h = Hypergraph(n=n, m=m, eptr=eptr, pins=pins.astype(np.int32), w=w)
    dh = to_device(h)
    R = rng.random(m).astype(np.float32)
    eta = rng.random(n).astype(np.float32)
    p = hef.Params(k=4, b=1, local_clustering=False)
    cl, nc, eo = hef.cluster_level(dh, p, torch.as_tensor(R, device="cuda"),
                                   torch.as_tensor(eta, device="cuda"),
                                   torch.zeros((n, 8), device="cuda"),
                                   torch.ones(8, dtype=torch.float64, device="cuda"))
    ref = ocl.cluster_level(n, m, h.eptr, h.pins, R, eta, None, np.ones(8), 0.5, False)
    assert nc == ref.n_clusters and np.array_equal(cl.cpu().numpy(), ref.label)
    assert np.array_equal(eo.cpu().numpy().view(np.uint32), ref.eta.view(np.uint32))
    cl, nc, _, _ = hef.coarsen(dh, hef.Params(k=20, b=2, levels=2))
    cl = cl.cpu().numpy()
    assert 0 < nc < n and cl.min() == 0 and np.unique(cl).size == nc


LAYOUTS = {"long": [1000] * 130, "giant": [3] * 70 + [13000] + [3] * 100,
           "long then short": [700] * 64 + [2] * 300, "short then long": [2] * 64 + [4096] * 3 + [9],
           "span": [4096], "below": [2] * 63 + [4096 - 126], "above": [2] * 63 + [4097 - 126]}


@pytest.mark.parametrize("layout", list(LAYOUTS))
def test_long_pin_ranges_are_split(layout):
    """64 hyperedges of more than 4096 pins are walked by several waves, which
    start at multiples of 4096 positions: bad pins at every start and end of
    such a span are found, every incidence carries its hyperedge, and a
    hyperedge is split if any of the waves sees it (whole-number sums, equal)."""
    say(f"case: long pin ranges {layout}")
    sizes = np.array(LAYOUTS[layout])
    m, n, nnz = len(sizes), 14000, int(sizes.sum())
    rng = np.random.default_rng(m)
    eptr = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    first = (rng.random(m) * (n - sizes)).astype(np.int64)
    pins = (np.repeat(first, sizes) + np.arange(nnz) - np.repeat(eptr[:-1], sizes)).astype(np.int32)
    w = rng.integers(1, 9, m).astype(np.float32)
    eid = np.repeat(np.arange(m), sizes)
    spans = [x * 4096 for x in range(1, nnz // 4096 + 1)]
    blocks = [int(eptr[b]) + 4096 for b in range(0, m, 64)] + [int(x) for x in eptr[64:m:64]]
    at = sorted({p + d for p in [0, nnz - 1] + spans + blocks for d in (-1, 0, 1) if 0 <= p + d < nnz})
    at = [j for j in at if j > eptr[eid[j]]]
    at = at if len(at) <= 40 else at[:10] + [at[i] for i in rng.choice(len(at), 30, replace=False)]
    label0 = torch.zeros(n, dtype=torch.int32, device="cuda")
    for j in at:
        p = pins.copy()
        p[j] = p[j - 1]
        with pytest.raises(hef.HefError, match="code 4"):
            hef.conductance(hef.DeviceHypergraph.from_arrays(n, m, eptr, p, w), label0, 1)
    h = Hypergraph(n=n, m=m, eptr=eptr, pins=pins, w=w)
    dh = to_device(h)
    # one node apart from the others, at the same places
    for j in at[:12]:
        label = np.zeros(n, np.int32)
        label[pins[j]] = 1
        cut, vol, _, _ = hef.conductance(dh, torch.as_tensor(label, device="cuda"), 2)
        k = float(w[eid[pins == pins[j]]].sum())
        assert cut.cpu().tolist() == [k, k]
        assert vol.cpu().tolist() == [float((w * sizes).sum()) - k, k]
    # every incidence: a value per hyperedge, summed at the nodes by the star operator
    x = torch.zeros((n + m, 1), device="cuda")
    x[n:, 0] = torch.arange(m, device="cuda") % 13
    y = hef.debug_apply(dh, 0, x).cpu().numpy()[:n, 0].astype(np.float64)
    alpha = np.sqrt(w.astype(np.float64)) / sizes
    db = np.bincount(pins, weights=np.repeat(w / sizes, sizes), minlength=n)
    ref = np.bincount(pins, weights=np.repeat(alpha * (np.arange(m) % 13), sizes), minlength=n)
    ref = np.where(db > 0, ref / np.sqrt(np.where(db > 0, db, 1.0)), 0.0)
    deg = np.bincount(pins, minlength=n).max()
    assert np.abs(y - ref).max() <= (deg + 4) * 2.0 ** -24 * max(np.abs(ref).max(), 1.0)


@pytest.mark.parametrize("k,b", [(5, 1), (8, 4), (9, 4), (17, 8)])
@pytest.mark.parametrize("many", [2048, 2049])
def test_many_long_hyperedges(many, k, b):
    """Up to 2048 hyperedges of more than 32 pins each take a workgroup in the
    ratios and in their adjoint, more than that only those above 128 pins; with
    lane groups of 32 lanes and more every one in the ratios, those above 64 in
    the adjoint.  As many fours of pins as lane groups and fewer, whole and not.  Ratios
    against float64 on the pool (bounds as in test_long_hyperedge_ratios), the
    gradient against the float64 autograd oracle at the adjoint tests' 1e-3."""
    from oracle import gradient as ogr
    from oracle import resistance as orr
    from tests.gpu_common import starts
    say(f"case: many long hyperedges {many} k={k} b={b}")
    special = [127, 128, 129, 130, 255, 300, 513, 36, 37, 63, 64, 65, 66]
    sizes = special + [33 + i % 4 for i in range(many - len(special))] + _mixed_sizes(300, 3) + [32]
    assert sum(s > 32 for s in sizes) == many
    w = np.random.default_rng(2).uniform(0.5, 2.0, len(sizes)).astype(np.float32)
    h = _hg(9000, sizes, 5, w)
    dh = to_device(h)
    Xs, Xc, xs, xc = starts(h, b)
    R, qh, chi = hef.resistance(dh, hef.Params(k=k, b=b), xs, xc, return_pool=True)
    s = orr.edge_spread(h.eptr, h.pins, chi.cpu().double().numpy())
    q = h.w.astype(np.float64) @ s
    assert np.abs(qh.cpu().numpy() - q).max() <= 2 * h.m * 2.0 ** -53 * q.max()
    np.testing.assert_allclose(R.cpu().numpy(), (s / q[None, :]).max(1), rtol=2.0 ** -22, atol=0)
    coef = np.random.default_rng(3).standard_normal(h.m).astype(np.float32)
    _, ref, _ = ogr.loss_and_grad(h.n, h.m, h.eptr, h.pins, h.w, Xs, Xc, k, coef)
    dw = hef.resistance_backward(dh, hef.Params(k=k, b=b), torch.as_tensor(coef, device="cuda"),
                                 xs, xc).cpu().numpy()
    assert np.linalg.norm(dw - ref) <= 1e-3 * np.linalg.norm(ref)


@pytest.mark.parametrize("together", [1, 3, 4, 64])
@pytest.mark.parametrize("length", [256, 257, 321, 640])
def test_long_segments_side_by_side(together, length):
    """Nodes of `length` hyperedges and hyperedges of `length` pins, so many of
    them among 64 neighbours: up to three times the longest's terms the wave
    takes them above 256, else a lane each.  Eq. (15) sums eta in pin order
    either way (bit for bit); the node scales through the star operator, with
    (degree + 4) roundings of relative 2^-24."""
    from oracle import clustering as ocl
    say(f"case: long segments side by side {together} of {length}")
    n, gap = 4000, {1: 64, 3: 20, 4: 16, 64: 1}[together]
    rng = np.random.default_rng(together + length)
    long_at = [(64 + gap * i, length + (i % 2)) for i in range(together)]
    h = _hg(n, _mixed_sizes(300, length, long_at), length + together)
    hubs = 128 + gap * np.arange(together)
    others = 1000 + np.array([rng.choice(n - 1000, length, replace=False) for _ in hubs])
    extra = np.stack([np.repeat(hubs, length), others.reshape(-1)], 1)
    eptr = np.concatenate([h.eptr, h.eptr[-1] + 2 * np.arange(1, len(extra) + 1)])
    pins = np.concatenate([h.pins, extra.reshape(-1)]).astype(np.int32)
    m = len(eptr) - 1
    w = rng.uniform(0.5, 2.0, m).astype(np.float32)
    h = Hypergraph(n=n, m=m, eptr=eptr, pins=pins, w=w)
    dh = to_device(h)
    R = (rng.random(m) * 10.0 ** rng.integers(-3, 3, m)).astype(np.float32)
    eta = (rng.random(n) * 10.0 ** rng.integers(-6, 3, n)).astype(np.float32)
    cl, nc, eo = hef.cluster_level(dh, hef.Params(k=4, b=1, local_clustering=False, percentile=1.0),
                                   torch.as_tensor(R, device="cuda"),
                                   torch.as_tensor(eta, device="cuda"),
                                   torch.zeros((n, 8), device="cuda"),
                                   torch.ones(8, dtype=torch.float64, device="cuda"))
    ref = ocl.cluster_level(n, m, eptr, pins, R, eta, None, np.ones(8), 1.0, False)
    assert nc == ref.n_clusters and np.array_equal(cl.cpu().numpy(), ref.label)
    assert np.array_equal(eo.cpu().numpy().view(np.uint32), ref.eta.view(np.uint32))
    x = torch.zeros((n + m, 1), device="cuda")
    x[n:, 0] = torch.arange(m, device="cuda") % 13
    y = hef.debug_apply(dh, 0, x).cpu().numpy()[:n, 0].astype(np.float64)
    sizes = np.diff(eptr)
    alpha = np.sqrt(w.astype(np.float64)) / sizes
    db = np.bincount(pins, weights=np.repeat(w / sizes, sizes), minlength=n)
    r = np.bincount(pins, weights=np.repeat(alpha * (np.arange(m) % 13), sizes), minlength=n)
    r = np.where(db > 0, r / np.sqrt(np.where(db > 0, db, 1.0)), 0.0)
    deg = np.bincount(pins, minlength=n).max()
    assert np.abs(y - r).max() <= (deg + 4) * 2.0 ** -24 * max(np.abs(r).max(), 1.0)


@pytest.mark.parametrize("order", ["up", "down", "mixed"])
def test_attach_chain(order):
    """A chain of 1500 isolated nodes that each pick the next (gaps that
    shrink), numbered along it, against it and at random, beside short chains:
    the union-find joins it to one cluster; the level against the oracle, bit
    for bit."""
    from oracle import clustering as ocl
    say(f"case: attach chain {order}")
    L, n = 1500, 2400
    at = np.cumsum(np.linspace(2, 1, L))
    rng = np.random.default_rng(6)
    pos = np.concatenate([at, 4000 + np.sort(rng.uniform(0, 4000, n - L))]).astype(np.float32)
    num = {"up": np.arange(n), "down": np.arange(n)[::-1], "mixed": rng.permutation(n)}[order]
    edges = np.stack([num[:-1], num[1:]], 1)
    edges = np.delete(edges, L - 1, 0)  # (the chain is a component of its own)
    m = len(edges)
    eptr, pins = 2 * np.arange(m + 1), np.sort(edges, 1).reshape(-1).astype(np.int32)
    chi = np.zeros((n, 8), np.float32)
    chi[num, 3] = pos
    qh = np.ones(8)
    R = np.ones(m, np.float32)  # none below the threshold: every node is isolated
    h = Hypergraph(n=n, m=m, eptr=eptr.astype(np.int64), pins=pins, w=np.ones(m, np.float32))
    cl, nc, eo = hef.cluster_level(to_device(h), hef.Params(k=4, b=1),
                                   torch.as_tensor(R, device="cuda"), None,
                                   torch.as_tensor(chi, device="cuda"),
                                   torch.as_tensor(qh, device="cuda"))
    ref = ocl.cluster_level(n, m, h.eptr, h.pins, R, None, chi, qh, 0.5, True)
    chain = np.unique(ref.label[num[:L]])
    assert len(chain) < L / 20  # (float32 positions may tie a few gaps)
    assert nc == ref.n_clusters and np.array_equal(cl.cpu().numpy(), ref.label)
    assert np.array_equal(eo.cpu().numpy().view(np.uint32), ref.eta.view(np.uint32))


@pytest.mark.parametrize("scale", [1.0, 1e-6, 3e4])
@pytest.mark.parametrize("K", [8, 40, 160])
def test_best_neighbour_on_smooth_vectors(K, scale):
    """Pools whose rows differ little against their entries, in entries from
    float16's subnormal range to near its largest: the screen's error bounds
    decide which candidates get their exact distance.  The level against the
    oracle, bit for bit."""
    from oracle import clustering as ocl
    side = 40
    say(f"case: smooth vectors K={K} scale={scale}")
    n = side * side
    x = np.arange(side) / side
    modes = [(i, j) for i in range(16) for j in range(16)][1:K + 1]
    chi = np.stack([np.outer(np.cos(np.pi * i * x), np.cos(np.pi * j * x)).reshape(-1)
                    for i, j in modes], 1)
    chi = (scale * chi).astype(np.float32)
    qh = np.array([0.1 * (i * i + j * j) for i, j in modes])
    g = np.arange(n).reshape(side, side)
    e = np.stack([g[a:a + 3, b:b + 3].reshape(-1) for a in range(side - 2)
                  for b in range(0, side - 2, 2)])
    m = len(e)
    h = Hypergraph(n=n, m=m, eptr=9 * np.arange(m + 1), pins=e.reshape(-1).astype(np.int32),
                   w=np.ones(m, np.float32))
    R = np.random.default_rng(K).random(m).astype(np.float32)
    for pct in (1e-6, 0.3):
        out = hef.cluster_level(to_device(h), hef.Params(k=K // 2, b=1, percentile=pct),
                                torch.as_tensor(R, device="cuda"), None,
                                torch.as_tensor(chi, device="cuda"),
                                torch.as_tensor(qh, device="cuda"))
        ref = ocl.cluster_level(n, m, h.eptr, h.pins, R, None, chi, qh, pct, True)
        assert out[1] == ref.n_clusters and np.array_equal(out[0].cpu().numpy(), ref.label)
        assert np.array_equal(out[2].cpu().numpy().view(np.uint32), ref.eta.view(np.uint32))


def _hub(n, deg, size, seed, pool=None, hub=0):
    """Node `hub` in `deg` hyperedges of `size` pins drawn from `pool`, and one
    hyperedge apart."""
    rng = np.random.default_rng(seed)
    pool = np.setdiff1d(np.arange(n), [hub]) if pool is None else np.asarray(pool)
    step = rng.integers(1, max(2, len(pool) // size), deg)
    draw = (rng.integers(0, len(pool), deg)[:, None] + step[:, None] * np.arange(size - 1)) % len(pool)
    edges = [np.sort(np.append(pool[d], hub)) for d in draw]
    edges.insert(deg // 2, np.array([1, 2, 3]))
    eptr = np.concatenate([[0], np.cumsum([len(e) for e in edges])]).astype(np.int64)
    w = rng.uniform(0.5, 2.0, len(edges)).astype(np.float32)
    return Hypergraph(n=n, m=len(edges), eptr=eptr, pins=np.concatenate(edges).astype(np.int32), w=w)


@pytest.mark.parametrize("deg,size", [(255, 4), (256, 3), (256, 4), (511, 3), (512, 8), (1100, 3),
                                      (3000, 5), (300, 200), (20000, 2)])
def test_rating_of_hubs(deg, size):
    """A node of 256 hyperedges or more is shared by waves, a range of hash
    classes each: one class and many, fewer waves than classes, hyperedges of
    less and of more pins than lanes, and repeated neighbours, whose terms
    must add up in hyperedge order."""
    from oracle import rating as orat
    say(f"case: rating hub deg={deg} size={size}")
    for n, pool in ((30000, None), (30000, np.arange(500, 500 + max(40, 2 * size)))):
        hg = _hub(n, deg, size, deg + size, pool, hub=7 if pool is None else n - 1)
        R = np.random.default_rng(5).uniform(0.01, 1.0, hg.m).astype(np.float32)
        for shift in (0.0, 1.0):
            best, val = hef.rating(to_device(hg), torch.as_tensor(R, device="cuda"), shift)
            nodes = np.unique(np.concatenate([[0, 1, 2, 7, n - 1], hg.pins[:40]]))
            rb, rv = orat.best_neighbours(hg.n, hg.m, hg.eptr, hg.pins, hg.w, R, shift, nodes)
            assert np.array_equal(best.cpu().numpy()[nodes], rb)
            assert np.array_equal(val.cpu().numpy()[nodes], rv)


def test_rating_of_hubs_with_full_tables():
    """Neighbours that all fall in one class of the first sweep overflow its
    table, which is halved until they fit; and many hubs at once."""
    from oracle import rating as orat
    say("case: rating hubs, full tables and many hubs")
    n = 400000
    q = np.arange(8, n, dtype=np.uint64)
    hsh = (q * 2654435769) & 0xFFFFFFFF
    pool = q[((hsh >> 19) & 7) == 5].astype(np.int64)[:6000]  # one of 8 classes below 10 bits
    hg = _hub(n, 3000, 3, 3, pool)
    R = np.random.default_rng(5).uniform(0.01, 1.0, hg.m).astype(np.float32)
    best, val = hef.rating(to_device(hg), torch.as_tensor(R, device="cuda"), 0.0)
    nodes = np.unique(np.concatenate([[0, 1, 2], hg.pins[:30]]))
    rb, rv = orat.best_neighbours(hg.n, hg.m, hg.eptr, hg.pins, hg.w, R, 0.0, nodes)
    assert np.array_equal(best.cpu().numpy()[nodes], rb)
    assert np.array_equal(val.cpu().numpy()[nodes], rv)
    n, m = 700, 90000  # every node in about 390 hyperedges
    rng = np.random.default_rng(9)
    pins = np.sort(np.stack([3 * rng.choice(n // 3, m), 3 * rng.choice(n // 3, m) + 1,
                             3 * rng.choice(n // 3, m) + 2], 1), 1).reshape(-1)
    hg = Hypergraph(n=n, m=m, eptr=3 * np.arange(m + 1), pins=pins.astype(np.int32),
                    w=rng.uniform(0.5, 2.0, m).astype(np.float32))
    R = rng.uniform(0.01, 1.0, m).astype(np.float32)
    best, val = hef.rating(to_device(hg), torch.as_tensor(R, device="cuda"), 0.0)
    nodes = np.arange(0, n, 23)
    rb, rv = orat.best_neighbours(hg.n, hg.m, hg.eptr, hg.pins, hg.w, R, 0.0, nodes)
    assert np.array_equal(best.cpu().numpy()[nodes], rb)
    assert np.array_equal(val.cpu().numpy()[nodes], rv)


@pytest.mark.parametrize("nnz", [4095, 4096, 4097, 8191, 8192, 8193, 16385, 70001, 1048575, 1048576,
                                 1048577, 1052673])
def test_sorts_of_exact_sizes(nnz):
    """The incidence and label sorts at exactly the counts where they change:
    4 or 8 items a thread in one workgroup (4096), several workgroups (8192),
    tiles of 1024 or 4096 items (2^20); ids of 8, 16, 17 and 20 bits, i.e. one
    to three digits of 8 bits or two of 9.  Every node's degree from the
    conductance of single-node clusters (whole numbers), its hyperedges from the
    star operator."""
    say(f"case: exact sort sizes nnz={nnz}")
    for n in (200, 60000, 70000, 600000):
        rng = np.random.default_rng(nnz + n)
        m = nnz // 3
        sizes = np.full(m, 3)
        sizes[rng.permutation(m)[:nnz - 3 * m]] += 1
        eptr = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
        assert eptr[-1] == nnz
        first = rng.integers(0, n - 40, m)
        pins = np.repeat(first, sizes) + 11 * (np.arange(nnz) - np.repeat(eptr[:-1], sizes))
        h = Hypergraph(n=n, m=m, eptr=eptr, pins=pins.astype(np.int32), w=np.ones(m, np.float32))
        dh = to_device(h)
        deg = np.bincount(pins, minlength=n).astype(np.float64)
        perm = rng.permutation(n).astype(np.int32)
        cut, vol, _, _ = hef.conductance(dh, torch.as_tensor(perm, device="cuda"), n)
        assert np.array_equal(vol.cpu().numpy()[perm], deg)
        assert np.array_equal(cut.cpu().numpy()[perm], deg)
        x = torch.zeros((n + m, 1), device="cuda")
        x[n:, 0] = torch.arange(m, device="cuda") % 13
        y = hef.debug_apply(dh, 0, x).cpu().numpy()[:n, 0].astype(np.float64)
        db = np.bincount(pins, weights=np.repeat(1.0 / sizes, sizes), minlength=n)
        ref = np.bincount(pins, weights=np.repeat((np.arange(m) % 13) / sizes, sizes), minlength=n)
        ref = np.where(db > 0, ref / np.sqrt(np.where(db > 0, db, 1.0)), 0.0)
        assert np.abs(y - ref).max() <= (deg.max() + 4) * 2.0 ** -24 * max(np.abs(ref).max(), 1.0)


@pytest.mark.parametrize("m", [4096, 4097, 8192, 8193, 1048576, 1048577])
def test_level_order_at_sort_sizes(m):
    """The 32-bit sort of the updated resistances (four digits) at the same
    counts, with many equal values, whose order is the hyperedges': the
    contraction of one level against the oracle."""
    from oracle import clustering as ocl
    n = 3 * m // 2
    say(f"case: level order m={m}")
    rng = np.random.default_rng(m)
    first = rng.integers(0, n - 9, m)
    pins = np.stack([first, first + rng.integers(1, 9, m)], 1).reshape(-1).astype(np.int32)
    h = Hypergraph(n=n, m=m, eptr=2 * np.arange(m + 1), pins=pins, w=np.ones(m, np.float32))
    R = (rng.integers(1, 1 + m // 4, m) * np.float32(2.0) ** rng.integers(-90, 20, m)).astype(np.float32)
    cl, nc, _ = hef.cluster_level(to_device(h), hef.Params(k=4, b=1, local_clustering=False),
                                  torch.as_tensor(R, device="cuda"), None,
                                  torch.zeros((n, 8), device="cuda"),
                                  torch.ones(8, dtype=torch.float64, device="cuda"))
    owner, _ = ocl.greedy_contract(n, h.eptr, h.pins, R, ocl.threshold(R, 0.5))
    prov = np.arange(n)
    taken = owner >= 0
    prov[taken] = pins[2 * owner[taken]]
    roots = np.unique(prov)
    assert nc == len(roots) and np.array_equal(cl.cpu().numpy(), np.searchsorted(roots, prov))
