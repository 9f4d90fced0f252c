"""fp32 products on the bf16 matrix cores (three-plane split): statistics and
preconditioning at the edges of tiles, stages and accumulation runs, on
contiguous and on oddly strided (unaligned) views, against fp64 products of
the same inputs, and the handling of infinities, NaN and values that round up
to infinity in bf16.

Bound, per output element with s = sum |a||b| (fp64): a 16-deep step rounds
at most 12 times at a magnitude of at most s; over the first 256 k ten of the
twelve only at the magnitude of the smaller products (below 2^-7 s), later
runs of 256 k are added once each; the dropped products are at most 2^-24 s, and
the products that an instruction cuts are below 2^-23 of a larger one of the same
group of eight (seven per group, in one group of the whole sum at that size):
  |err| <= (2.1 steps(min(K, 256)) + [K > 256] (192 + K / 256) + 5) 2^-24 s.
"""
import numpy as np
import pytest

from tests.gpu_util import gpu_env, host, say, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    torch, B, dev = gpu_env()
    h = B.shampoo_create(0)
    yield torch, B, dev, h
    B.shampoo_destroy(h)


def _view(torch, dev, x, pad, off, dtype):
    """x as a view with row stride cols + pad, starting `off` elements into its buffer."""
    m, n = x.shape
    buf = torch.zeros(off + m * (n + pad), device=dev, dtype=dtype)
    v = buf[off:].view(m, n + pad)[:, :n]
    v.copy_(to_dev(torch, x, dev))
    return v


def _bound(K, s):
    units = 2.1 * -(-min(K, 256) // 16) + (192 + K / 256 if K > 256 else 0) + 5
    return units * 2.0 ** -24 * s + 1e-37


SIZES = [(1, 1), (1, 300), (3, 17), (16, 16), (31, 33), (127, 15), (128, 16), (129, 257), (130, 256), (257, 130),
         (200, 513)]


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("pad,off", [(0, 0), (3, 1)])
def test_stats_edges(env, bf16, pad, off):
    torch, B, dev, h = env
    dt = torch.bfloat16 if bf16 else torch.float32
    r = np.random.default_rng(7)
    blocks, want = [], []
    for m, n in SIZES:
        g = (r.standard_normal((m, n)) * np.exp(r.uniform(-6, 6, (m, 1)))).astype(np.float32)
        G = _view(torch, dev, g, pad, off, dt)
        x = host(G.float().contiguous()).astype(np.float64)
        L = torch.zeros(m, m, device=dev)
        R = torch.zeros(n, n, device=dev)
        blocks.append(B.Block(G=G, L=L, R=R))
        want.append(x)
    say(f"stats edges bf16={bf16} pad={pad}")
    B.shampoo_update_stats(h, blocks)
    torch.cuda.synchronize()
    for b, x in zip(blocks, want):
        for got, a in ((b.L, x), (b.R, x.T)):
            got = host(got).astype(np.float64)
            assert np.array_equal(got, got.T)
            share = float((np.abs(got - a @ a.T) / _bound(a.shape[1], np.abs(a) @ np.abs(a).T)).max())
            assert share <= 1.0, (x.shape, share)


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("pad,off", [(0, 0), (3, 1)])
def test_precondition_edges(env, bf16, pad, off):
    torch, B, dev, h = env
    dt = torch.bfloat16 if bf16 else torch.float32
    r = np.random.default_rng(11)
    blocks, want = [], []
    for i, (m, n) in enumerate(SIZES):
        G = _view(torch, dev, r.standard_normal((m, n)).astype(np.float32), pad, off, dt)
        P = _view(torch, dev, np.zeros((m, n), np.float32), pad, off, torch.float32)
        left, right = [(True, True), (True, False), (False, True)][i % 3]
        l, q = (0.5 * (a + a.T) for a in (r.standard_normal((m, m)), r.standard_normal((n, n))))
        Lr = to_dev(torch, l.astype(np.float32), dev) if left else None
        Rr = to_dev(torch, q.astype(np.float32), dev) if right else None
        blocks.append(B.Block(G=G, P=P, Lr=Lr, Rr=Rr))
    say(f"precondition edges bf16={bf16} pad={pad}")
    B.shampoo_precondition(h, blocks)
    torch.cuda.synchronize()
    for b in blocks:
        x = host(b.G.float().contiguous()).astype(np.float64)
        m, n = x.shape
        s = np.abs(x)
        bound = np.zeros_like(x)
        if b.Rr is not None:
            q = host(b.Rr).astype(np.float64)
            bound = _bound(n, s @ np.abs(q)) + 2.0 ** -24 * (s @ np.abs(q))
            x, s = x @ q, s @ np.abs(q)
        if b.Lr is not None:
            l = host(b.Lr).astype(np.float64)
            bound = np.abs(l) @ bound + _bound(m, np.abs(l) @ s)
            x = l @ x
        share = float((np.abs(host(b.P.contiguous()).astype(np.float64) - x) / bound).max())
        assert share <= 1.0, (x.shape, share)


@pytest.mark.parametrize("m,count", [(96, 1), (96, 90)])
def test_long_contractions(env, m, count):
    """Error of long sums in the norm and on the diagonal of a Gram matrix (few
    tiles and many): each output is a sum of K / 256 runs, which round at the
    magnitude of the sum once each and inside at that of a run, 32 times
    (sqrt(32) / 2 units of 2^-24 of the run, as independent roundings): below
    sqrt(K / 256) / 2 + sqrt(32) / 2 + 2 units, 6.9 at K = 4096 (measured 1.6 to
    3.5).  Losing the products of order 2^-16 of one run costs 30 units in the
    norm at K = 513 and 16 at 1024 (emulated); the element bound would pass."""
    torch, B, dev, h = env
    r = np.random.default_rng(m)
    for K in (257, 513, 1024, 4096):
        g = r.standard_normal((m, K)).astype(np.float32)
        q = r.standard_normal((K, K)) if K < 4096 else np.zeros((K, K))
        q = (0.5 * (q + q.T)).astype(np.float32)
        G, Q = to_dev(torch, g, dev), to_dev(torch, q, dev)
        Ls = [torch.zeros(m, m, device=dev) for _ in range(count)]
        P = torch.zeros(m, K, device=dev)
        say(f"long contraction m={m} count={count} K={K}")
        B.shampoo_update_stats(h, [B.Block(G=G, L=L) for L in Ls])
        B.shampoo_precondition(h, [B.Block(G=G, P=P, Rr=Q)])
        x = g.astype(np.float64)
        units = np.sqrt(K / 256) / 2 + np.sqrt(32) / 2 + 2
        want = x @ x.T
        for L in (Ls[0], Ls[-1]):
            got = host(L).astype(np.float64)
            assert np.linalg.norm(got - want) <= units * 2.0 ** -24 * np.linalg.norm(want), K
            d = np.diagonal(got) / np.diagonal(want) - 1
            assert np.sqrt((d ** 2).mean()) <= units * 2.0 ** -24, K
        if K < 4096:
            want = x @ q.astype(np.float64)
            assert np.linalg.norm(host(P) - want) <= units * 2.0 ** -24 * np.linalg.norm(want), K


@pytest.mark.parametrize("m,n", [(40, 70), (300, 200)])
def test_non_finite(env, m, n):
    """An output is what the fp32 sum gives: infinite or NaN only where an
    infinity, a NaN or an overflow enters it, finite elsewhere."""
    torch, B, dev, h = env
    r = np.random.default_rng(3)
    g = r.uniform(0.5, 1.0, (m, n)).astype(np.float32)
    g[1, 2] = np.inf
    g[m - 1, 5] = np.nan
    g[7, n - 1] = 3.4e38  # rounds to infinity in bf16
    G = to_dev(torch, g, dev)
    L, R = torch.zeros(m, m, device=dev), torch.zeros(n, n, device=dev)
    say(f"non-finite {m}x{n}")
    B.shampoo_update_stats(h, [B.Block(G=G, L=L, R=R)])
    torch.cuda.synchronize()
    x = g.astype(np.float64)
    for got, a in ((L, x), (R, x.T)):
        want = a @ a.T
        want[np.abs(want) > 3.5e38] = np.inf  # the largest finite sum here is about 3.4e38
        got = host(got).astype(np.float64)
        assert np.array_equal(np.isnan(got), np.isnan(want))
        assert np.array_equal(np.isinf(got), np.isinf(want))
        f = np.isfinite(want)
        share = float((np.abs(got[f] - want[f]) / (1e-5 * np.abs(want[f]))).max())
        assert share <= 1.0, share


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("m,n,pad", [(1, 1, 0), (33, 31, 1), (128, 128, 0), (129, 300, 3), (257, 64, 0), (300, 520, 0)])
def test_few_tiles_same_bits(env, m, n, pad, bf16):
    """A block alone (few tiles: one wave per 32 x 32 block) and the same
    block in a launch of many tiles (128 x 128 workgroups): statistics,
    preconditioning and the fused graft agree bit for bit, with a non-finite
    gradient entry in one of the statistics."""
    torch, B, dev, h = env
    dt = torch.bfloat16 if bf16 else torch.float32
    r = np.random.default_rng(100 * m + n)
    g = r.standard_normal((m, n)).astype(np.float32)
    l, q = (to_dev(torch, (0.5 * (a + a.T)).astype(np.float32), dev)
            for a in (r.standard_normal((m, m)), r.standard_normal((n, n))))

    def block(left, right, x):
        t = dict(G=_view(torch, dev, x, pad, pad, dt))
        for k, v in (("W", 1.0), ("D", 0.5), ("P", 0.0)):
            t[k] = _view(torch, dev, np.full((m, n), v, np.float32), pad, 0, torch.float32)
        return B.Block(L=torch.ones(m, m, device=dev), R=torch.ones(n, n, device=dev), Lr=l if left else None,
                       Rr=q if right else None, **t)

    big = torch.zeros(1024, 1536, device=dev, dtype=dt)
    eye, eyn = torch.eye(1024, device=dev), torch.eye(1536, device=dev)
    say(f"few tiles {m}x{n} pad={pad} bf16={bf16}")
    for left, right in ((True, True), (True, False), (False, True)):
        x = g.copy()
        x[m // 2, n // 3] = np.inf if left and right else 0.25
        fill = B.Block(G=big, W=torch.zeros(1024, 1536, device=dev), D=torch.zeros(1024, 1536, device=dev),
                       P=torch.zeros(1024, 1536, device=dev), L=torch.zeros(1024, 1024, device=dev),
                       R=torch.zeros(1536, 1536, device=dev), Lr=eye if left else None, Rr=eyn if right else None)
        got = []
        for extra in ([], [fill]):
            b = block(left, right, x)
            norms = torch.zeros(3 * (1 + len(extra)), device=dev)
            B.shampoo_update_stats(h, [b] + extra, beta2=0.9)
            b.G[m // 2, n // 3] = 0.25
            B.shampoo_precondition_graft(h, [b] + extra, 0.05, norms=norms)
            torch.cuda.synchronize()
            got.append([host(v.contiguous()) for v in (b.L, b.R, b.P, b.D, b.W, norms[:3])])
        for a, c, what in zip(*got, ("L", "R", "P", "D", "W", "norms")):
            assert np.array_equal(a, c, equal_nan=True), (what, left, right)


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("m", [200, 1700])
def test_short_contractions(env, m, bf16):
    """Contractions of 1 to 33 with one column 30 times the others, alone
    (few tiles; the statistics of 1700 rows are many).  Up to 16 the sums are
    formed in fp64 and rounded once (2^-24 of the result, and 2^-48 s for the
    sum itself); above, they are within K 2^-24 s, one rounding per product."""
    torch, B, dev, h = env
    dt = torch.bfloat16 if bf16 else torch.float32
    r = np.random.default_rng(m)
    for K in (1, 2, 3, 4, 5, 12, 15, 16, 17, 33):
        g = r.standard_normal((m, K))
        g[:, K // 2] *= 30
        G = to_dev(torch, g.astype(np.float32), dev).to(dt)
        x = host(G.float()).astype(np.float64)
        L, R = torch.zeros(m, m, device=dev), torch.zeros(K, K, device=dev)
        q = r.standard_normal((K, K))
        q = (0.5 * (q + q.T)).astype(np.float32)
        P, Pt = torch.zeros(m, K, device=dev), torch.zeros(K, m, device=dev)
        Q, Gt = to_dev(torch, q, dev), G.T.contiguous()
        say(f"short contraction m={m} K={K} bf16={bf16}")
        B.shampoo_update_stats(h, [B.Block(G=G, L=L, R=R)])
        B.shampoo_precondition(h, [B.Block(G=G, P=P, Rr=Q)])
        B.shampoo_precondition(h, [B.Block(G=Gt, P=Pt, Lr=Q)])
        q = q.astype(np.float64)
        for got, a, b in ((L, x, x.T), (P, x, q), (Pt, q, x.T)):
            got, want = host(got).astype(np.float64), a @ b
            s = np.abs(a) @ np.abs(b)
            bound = 2.0 ** -24 * np.abs(want) + 2.0 ** -48 * s if a.shape[1] <= 16 else K * 2.0 ** -24 * s
            assert (np.abs(got - want) <= bound).all(), (K, a.shape)


@pytest.mark.parametrize("exp", [-140, -126, -115, -108, 40, 55])
@pytest.mark.parametrize("m,n", [(60, 100), (260, 700)])
def test_tiny_and_huge_elements(env, m, n, exp):
    """Gradients around 2^exp keep the accuracy of ordinary ones (the bound of
    the edge tests; subnormal inputs are exact, so nothing is added for them):
    P with roots around 2^60 (normal results) for the tiny ones and 1 for the
    huge ones, whose statistics reach 2^120, and the statistics of tiny rows
    beside rows around 1."""
    torch, B, dev, h = env
    r = np.random.default_rng(n)
    g = r.standard_normal((m, n)) * 2.0 ** exp
    if exp < 0:
        g[::2] *= 2.0 ** -exp
    g = g.astype(np.float32)
    sc = 2.0 ** 60 if exp < 0 else 1.0
    l, q = ((0.5 * (a + a.T) * sc).astype(np.float32) for a in (r.standard_normal((m, m)), r.standard_normal((n, n))))
    tiny = g[1::2].copy()
    x, t = g.astype(np.float64), tiny.astype(np.float64)
    l = l[:len(t), :len(t)].copy()
    Tt = to_dev(torch, tiny, dev)
    L = torch.zeros(m, m, device=dev)
    P, Q = (torch.zeros(*t.shape, device=dev) for _ in range(2))
    say(f"elements around 2^{exp}, {m}x{n}")
    B.shampoo_update_stats(h, [B.Block(G=to_dev(torch, g, dev), L=L)])
    B.shampoo_precondition(h, [B.Block(G=Tt, P=P, Lr=to_dev(torch, l, dev)), B.Block(G=Tt, P=Q, Rr=to_dev(torch, q, dev))])
    l, q = l.astype(np.float64), q.astype(np.float64)
    for got, a, b in ((L, x, x.T), (P, l, t), (Q, t, q)):
        got, want, s = host(got).astype(np.float64), a @ b, np.abs(a) @ np.abs(b)
        ok = np.abs(got - want) <= _bound(a.shape[1], s) - 1e-37 + 2.0 ** -148
        assert ok.all(), (a.shape, float((np.abs(got - want) / s).max()))


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("m,n", [(16, 130), (130, 5), (1, 260)])
def test_short_contractions_of_many_blocks(env, m, n, bf16):
    """90 blocks with a short side (launches of many tiles, both sides and each)
    against every block alone: statistics, P, the fused graft's P, D, W and norms
    bit for bit."""
    torch, B, dev, h = env
    dt = torch.bfloat16 if bf16 else torch.float32
    r = np.random.default_rng(m)
    say(f"many short blocks {m}x{n} bf16={bf16}")
    l, q = (0.5 * (a + a.T).astype(np.float32) for a in (r.standard_normal((m, m)), r.standard_normal((n, n))))
    ld, qd = to_dev(torch, l, dev), to_dev(torch, q, dev)
    G = [to_dev(torch, r.standard_normal((m, n)).astype(np.float32), dev).to(dt) for _ in range(5)]

    def run(idx, left, right):
        f = lambda v, a=m, b=n: torch.full((a, b), v, device=dev)
        bl = [B.Block(G=G[i % 5], W=f(1.0), D=f(0.5), P=f(0.0), L=f(0.0, m, m), R=f(0.0, n, n),
                      Lr=ld if left else None, Rr=qd if right else None) for i in idx]
        norms = torch.zeros(3 * len(bl), device=dev)
        B.shampoo_update_stats(h, bl)
        B.shampoo_precondition(h, bl)
        plain = [host(b.P) for b in bl]
        B.shampoo_precondition_graft(h, bl, 0.05, norms=norms)
        nm = host(norms).reshape(-1, 3)
        return [[plain[i], host(b.P), host(b.D), host(b.W), host(b.L), host(b.R), nm[i]] for i, b in enumerate(bl)]

    for left, right in ((True, True), (True, False), (False, True)):
        alone = [run([i], left, right)[0] for i in range(5)]
        for i, got in enumerate(run(range(90), left, right)):
            for k, (x, y) in enumerate(zip(got, alone[i % 5])):
                assert np.array_equal(x, y), (i, k, left, right)
            assert np.array_equal(got[0], got[1])


def _overflow(x):
    """fp64 products as an fp32 result holds them (no sum here is near the limit)."""
    return np.where(np.abs(x) > 3.5e38, np.sign(x) * np.inf, x)


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("left,right", [(True, True), (True, False), (False, True)])
@pytest.mark.parametrize("m,n", [(9, 14), (40, 70), (300, 520)])
def test_non_finite_preconditioning(env, m, n, left, right, bf16):
    """P of gradients with an infinity, a NaN and a value that rounds up to
    infinity in bf16 (its bf16 form is the largest finite bf16): infinite or
    NaN, with the infinity's sign, exactly where the fp32 sums are, and
    accurate elsewhere; from the separate and the fused call, alone (few
    tiles) and in a launch of many tiles, the same bits.  Roots of one sign
    and 1e-3 in size keep the huge value's products finite."""
    torch, B, dev, h = env
    dt = torch.bfloat16 if bf16 else torch.float32
    r = np.random.default_rng(m)
    g = r.uniform(0.5, 1.0, (m, n)).astype(np.float32)
    g[1, 2], g[m - 1, 5], g[m // 2, n - 1], g[2, n // 2] = np.inf, np.nan, 3.4e38, -np.inf
    if bf16:
        g[m // 2, n - 1] = 3.38e38
    l, q = (1e-3 * a for a in (r.uniform(0.5, 1.0, (m, m)), r.uniform(0.5, 1.0, (n, n))))
    l, q = (0.5 * (a + a.T).astype(np.float32) for a in (l, q))
    G = to_dev(torch, g, dev).to(dt)
    x = host(G.float()).astype(np.float64)
    with np.errstate(invalid="ignore"):
        if right:
            x = _overflow(x @ q.astype(np.float64))
        if left:
            x = _overflow(l.astype(np.float64) @ x)

    def block(G, l, q):
        z = lambda: torch.zeros(G.shape[0], G.shape[1], device=dev)
        return B.Block(G=G, W=z(), D=z(), P=z(), Lr=l if left else None, Rr=q if right else None)

    ld, qd = to_dev(torch, l, dev), to_dev(torch, q, dev)
    big = torch.zeros(1024, 1536, device=dev, dtype=dt)
    fill = block(big, torch.eye(1024, device=dev), torch.eye(1536, device=dev))
    say(f"non-finite P {m}x{n} bf16={bf16} left={left} right={right}")
    got = []
    for extra in ([], [fill]):
        b = block(G, ld, qd)
        B.shampoo_precondition(h, [b] + extra)
        got.append(host(b.P))
        B.shampoo_precondition_graft(h, [b] + extra, 0.0)
        got.append(host(b.P))
    f = np.isfinite(x)
    assert f.any() or (left and right)
    for y in got:
        assert np.array_equal(y, got[0], equal_nan=True)
    y = got[0].astype(np.float64)
    assert np.array_equal(np.isnan(y), np.isnan(x)) and np.array_equal(y[np.isinf(x)], x[np.isinf(x)])
    assert (np.abs(y[f] - x[f]) <= 1e-5 * np.abs(x[f])).all()


@pytest.mark.parametrize("fill", ["one NaN", "one infinity", "all NaN", "all infinite"])
def test_non_finite_gradients_cost(env, fill):
    """A gradient that overflowed costs a small multiple of a finite one: the
    repair is at most one more pass on the fp32 instruction, 1.7 to 1.9 times the
    rest where every output takes it to the end (a loop in single lanes took 10
    to 100 times the finite call)."""
    torch, B, dev, h = env

    def timed(f):
        best = float("inf")
        for _ in range(4):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            f()
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b))
        return best

    n, count = 1024, 32
    z = lambda: [torch.zeros(n, n, device=dev) for _ in range(count)]
    G, W, D, P, L, R = ([torch.randn(n, n, device=dev) for _ in range(count)], *(z() for _ in range(5)))
    root = torch.eye(n, device=dev) + 0.01
    upd = B.PackedBlocks(h, [B.Block(G=G[i], W=W[i], D=D[i], P=P[i], Lr=root, Rr=root) for i in range(count)])
    sts = B.PackedBlocks(h, [B.Block(G=G[i], L=L[i], R=R[i]) for i in range(count)])
    run = lambda: (timed(lambda: B.shampoo_update_stats(h, sts)),
                   timed(lambda: B.shampoo_precondition_graft(h, upd, 0.0)))
    say(f"cost of non-finite gradients: {fill}")
    fine = run()
    for x in G:
        v = float("nan") if "NaN" in fill else float("inf")
        if "all" in fill:
            x.fill_(v)
        else:
            x[n // 3, n // 2] = v
    got = run()
    say(f"finite {fine[0]:.3f} {fine[1]:.3f} ms, {fill} {got[0]:.3f} {got[1]:.3f} ms")
    assert got[0] <= 4 * fine[0] and got[1] <= 4 * fine[1], (fine, got)
