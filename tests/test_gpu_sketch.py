"""GPU parity of the sketch-based boundary rule (inshr_quantize_sketch through the C ABI) against
oracle/sketch_kmeans.py on the same seeded inputs and the same uniform numbers.  Bit-exact:
classes, bucket counts, Lloyd rounds, boundaries, symbols, protected lists.  Centres: the clustering
is fp64 with the oracle's operation order except for the running sums of a draw (block scan against
a sequential sum), so the codebook is compared at 1e-6 relative and found equal in practice."""
import numpy as np
import pytest
import torch

from oracle import ref
from oracle import sketch_kmeans as sk

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_2306_11800_amd import api
    c = api.Context(torch.device("cuda:0"))
    yield c
    c.close()


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).to("cuda:0")


def families(rng, n):
    t3 = (rng.standard_t(3, n) * 0.015).astype(np.float32)
    zeros = t3.copy()
    zeros[rng.uniform(size=n) < 0.3] = 0.0
    zeros[rng.uniform(size=n) < 0.05] = -0.0
    positive = np.abs(t3) + np.float32(1e-3)
    wide = (np.exp(rng.uniform(-60, 60, n)) * rng.choice([-1.0, 1.0], n)).astype(np.float32)
    denormal = (rng.standard_normal(n) * 1e-40).astype(np.float32)
    denormal[::3] = t3[::3]
    lattice = (rng.integers(-5, 6, n) * 0.25).astype(np.float32)
    return dict(t3=t3, zeros=zeros, positive=positive, wide=wide, denormal=denormal, lattice=lattice)


def check(ctx, xs, cfgs, alpha, sigma, max_iter, seed):
    rng = np.random.default_rng(seed)
    uni = rng.uniform(size=(len(xs), 256))
    qs, info = ctx.quantize_sketch([dev(x) for x in xs], cfgs, uni, alpha=alpha, sigma=sigma,
                                   max_iter=max_iter)
    for i, (x, cfg) in enumerate(zip(xs, cfgs)):
        bits = cfg[0]
        K = 1 << bits
        base = ref.quantize(x, cfg)  # classes and thresholds of the exact-threshold oracle
        r = sk.quantize_values(x, base["sym"], K, alpha, sigma, uni[i], max_iter)
        q = qs[i]
        assert (q.n_pruned, q.n_outlier, q.n_kept) == (base["n_pruned"], base["n_outlier"], base["n_kept"])
        assert info[i] == (r["n_buckets"], r["rounds"]), (info[i], r["n_buckets"], r["rounds"])
        cb = q.codebook.cpu().numpy()[:K]
        np.testing.assert_allclose(cb, r["codebook"], rtol=1e-6, atol=0)
        assert np.array_equal(q.boundaries.cpu().numpy()[:K - 1].view(np.uint32), r["boundaries"].view(np.uint32))
        got = ref.unpack(q.packed.cpu().numpy().view(np.uint64), x.size, bits + 1)
        bad = np.nonzero(got != r["sym"])[0]
        assert bad.size == 0, (bad[:10], got[bad[:10]], r["sym"][bad[:10]])
        assert np.array_equal(q.outlier_idx.cpu().numpy().view(np.uint32), base["outlier_idx"])
        assert np.array_equal(q.outlier_val.cpu().numpy().view(np.uint32), base["outlier_val"].view(np.uint32))


def test_families_and_configurations(ctx):
    rng = np.random.default_rng(11)
    cfgs_all = [(2, 0, 0), (4, 100000, 1000), (8, 300000, 100), (3, 50000, 0), (8, 0, 1000)]
    for n in (1, 7, 1000, 16384 + 5, 70001):
        fam = families(rng, n)
        xs = list(fam.values())
        cfgs = [cfgs_all[(j + n) % len(cfgs_all)] for j in range(len(xs))]
        check(ctx, xs, cfgs, 0.01, 0.2, 100, 1000 + n)


def test_parameters(ctx):
    rng = np.random.default_rng(12)
    x = (rng.standard_t(3, 50000) * 0.015).astype(np.float32)
    for alpha, sigma, max_iter in ((0.01, 1.0, 100), (0.05, 0.0, 100), (0.5, 0.4, 100), (0.02, 0.2, 1),
                                   (0.02, 0.2, 0), (0.01, 0.1, 300)):
        check(ctx, [x, -np.abs(x)], [(5, 100000, 1000), (6, 0, 0)], alpha, sigma, max_iter, 7)


@pytest.mark.parametrize("m", [1, 64, 255, 256, 257, 384, 385, 512, 513, 768, 769, 1024, 1025, 1536, 1537, 4096, 4097, 8600])
def test_lists_of_every_length(ctx, m):
    """m non-empty buckets of both signs: the edges of what a lane keeps of them while the centres are drawn, of
    the lists in LDS and of those in device memory."""
    rng = np.random.default_rng(m)
    neg = m // 3
    mags = np.exp(0.0203 * (np.arange(m) - m // 2))
    x = np.repeat(np.concatenate([-mags[:neg], mags[neg:]]), rng.integers(1, 4, m)).astype(np.float32)
    check(ctx, [rng.permutation(x)], [(8 if m % 2 else 5, 0, 0)], 0.01, 0.2, 60, 2000 + m)


def running_sums(probs, m, per, waves):
    """The running sums that the draws compare with their target: `per` buckets to a lane, added in index order, the lanes'
    sums by a tree (in rows of 16, then rows, then halves), the waves' one after the other."""
    share = np.zeros(64 * waves * per)
    share[:m] = probs
    share = share.reshape(-1, per)
    upto = share[:, 0].copy()
    for q in range(1, per):
        upto = upto + share[:, q]
    out, base = np.zeros(64 * waves), 0.0
    for wv in range(waves):
        a = upto[64 * wv:64 * wv + 64].reshape(4, 16).copy()
        for step in (1, 2, 4, 8):
            a[:, step:] = a[:, step:] + a[:, :-step].copy()
        a[1] += a[0, 15]
        a[3] += a[2, 15]
        a[2:] += a[1, 15]
        out[64 * wv:64 * wv + 64] = base + a.ravel()
        base += a[3, 15]
    return out, upto, base


@pytest.mark.parametrize("m,per,waves", [(64, 4, 1), (300, 6, 1), (384, 6, 1), (700, 12, 1), (1000, 16, 1), (1500, 24, 1),
                                         (2000, 4, 8), (4000, 8, 8)])
def test_a_lane_whose_buckets_are_all_centres_is_not_drawn_from(ctx, m, per, waves):
    """The lanes' sums come from a tree, so a lane that adds nothing can still end an ulp above the lane before it.  The
    uniforms make every bucket of such a lane a centre and then aim at that ulp: the next centre is another one."""
    found = 0
    for seed in range(40):
        rng = np.random.default_rng(seed)
        mags = np.exp((0.0203 if m < 2000 else 0.0201) * (np.arange(m) - m // 2))
        x = np.repeat(np.concatenate([-mags[:m // 3], mags[m // 3:]]), rng.integers(1, 4, m)).astype(np.float32)
        sign, index, count = sk.sketch_histogram(x, 0.01)
        assert count.size == m
        xq = sk.bucket_value(sign, index, 0.01)
        w = sk.sample_weights(xq, count, 0.2)
        for lane in range(1, min(63, m // per - 1)):
            dist, uni = np.ones(m), []
            for b in range(lane * per, lane * per + per):
                sums, _, total = running_sums(dist * w, m, per, waves)
                p = dist * w
                uni.append((sums[lane - 1] + p[lane * per:b].sum() + 0.5 * p[b]) / total)
                d = (xq - xq[b]) ** 2
                dist = d if len(uni) == 1 else np.minimum(dist, d)
            sums, upto, total = running_sums(dist * w, m, per, waves)
            assert upto[lane] == 0.0
            top = sums[:lane].max()
            us = [top / total]
            us += [np.nextafter(us[0], 0.0), np.nextafter(us[0], 1.0)]
            us = [u for u in us if top <= u * total < sums[lane]]
            if us:
                found += 1
                uniforms = np.full((1, 256), 0.5)
                uniforms[0, :per + 1] = uni + us[:1]
                q, _ = ctx.quantize_sketch([dev(x)], [(5, 0, 0)], uniforms, alpha=0.01, sigma=0.2, max_iter=0)
                centres = q[0].codebook.cpu().numpy()[:32]
                assert np.isin(xq[lane * per:lane * per + per].astype(np.float32), centres).all()  # (as they were meant to be)
                assert np.unique(centres).size == 32, (seed, lane)
                break
        if found >= 3:
            break
    assert found


def test_sums_are_not_contracted(ctx):
    """Eleven symmetric buckets, four clusters, magnitude-only weights: after the first Lloyd round
    the two inner centres are exact mirror images only if every product is rounded before it is
    added (a fused multiply-add moves one of them by two ulps, the midpoint leaves zero, the zero
    bucket changes sides and a second round is counted)."""
    rng = np.random.default_rng(17)
    x = (rng.integers(-5, 6, 5000) * 0.25).astype(np.float32)
    check(ctx, [x], [(2, 0, 0)], 0.01, 0.0, 3, 5132)


def test_more_clusters_than_buckets(ctx):
    x = np.array([0.5, 0.5, -0.25, 0.0, 1.0, 1.0, 1.0, 0.5], np.float32)
    check(ctx, [x, np.full(300, 3.0, np.float32)], [(4, 0, 0), (8, 0, 0)], 0.01, 0.2, 50, 3)


def test_on_top_of_a_grid_search(ctx):
    rng = np.random.default_rng(14)
    xs = [(rng.standard_t(3, n) * 0.015).astype(np.float32) for n in (30000, 5, 16384, 50001)]
    grid = [(b, p, o) for b in (3, 6, 8) for p in (0, 200000) for o in (0, 1000)]
    cfgs = [grid[3], grid[0], grid[11], grid[6]]
    uni = rng.uniform(size=(len(xs), 256))
    dx = [dev(x) for x in xs]
    alone, info_a = ctx.quantize_sketch(dx, cfgs, uni)
    ctx.search(dx, grid, 0.01, want_scores=False)
    reuse, info_r = ctx.quantize_sketch(dx, cfgs, uni, reuse_search=True)
    assert info_a == info_r
    for a, r in zip(alone, reuse):
        assert torch.equal(a.packed, r.packed)
        assert torch.equal(a.codebook[:1 << a.bits], r.codebook[:1 << a.bits])
        assert torch.equal(a.boundaries[:(1 << a.bits) - 1], r.boundaries[:(1 << a.bits) - 1])
        assert torch.equal(a.outlier_idx, r.outlier_idx) and torch.equal(a.outlier_val, r.outlier_val)
    # without a matching search the call is refused
    from paper_2306_11800_amd import api
    with pytest.raises(api.InshrError) as e:
        ctx.quantize_sketch(dx[:2], cfgs[:2], uni[:2], reuse_search=True)
    assert e.value.code == -5


def check_search(ctx, xs, cfgs, eps, alpha, sigma, max_iter, seed, reuse_grid=None):
    rng = np.random.default_rng(seed)
    uni = rng.uniform(size=(len(xs), 256))
    dx = [dev(x) for x in xs]
    if reuse_grid is not None:
        ctx.search(dx, reuse_grid, eps, want_scores=False)
    qs, choices, info = ctx.search_sketch(dx, cfgs, uni, eps, alpha=alpha, sigma=sigma, max_iter=max_iter,
                                          reuse_search=reuse_grid is not None)
    for i, (x, cfg) in enumerate(zip(xs, cfgs)):
        base = ref.quantize(x, (8, cfg[1], cfg[2]))
        r = sk.search_bits(x, base["sym"], alpha, sigma, uni[i], max_iter, eps)
        ch = choices[i]
        assert abs(ch["sumsq"] - r["sumsq"]) <= 1e-6 * r["sumsq"]
        border = False
        for b in range(2, 9):
            want = r["sse"][b]
            assert abs(ch["sse"][b - 2] - want) <= 1e-6 * want + 1e-12 * r["sumsq"], (b, ch["sse"][b - 2], want)
            assert ch["rounds"][b - 2] == r["runs"][b]["rounds"]
            if r["sumsq"] > 0 and abs(want / r["sumsq"] - eps) <= 4e-6 * eps:
                border = True
        if border:
            continue
        assert (ch["best_bits"], ch["feasible"]) == (r["best_bits"], r["feasible"])
        bits = r["best_bits"]
        run = r["runs"][bits]
        q = qs[i]
        assert q.bits == bits and info[i][0] == run["n_buckets"]
        np.testing.assert_allclose(q.codebook.cpu().numpy(), run["codebook"], rtol=1e-6, atol=0)
        assert np.array_equal(q.boundaries.cpu().numpy().view(np.uint32), run["boundaries"].view(np.uint32))
        got = ref.unpack(q.packed.cpu().numpy().view(np.uint64), x.size, bits + 1)
        assert np.array_equal(got, run["sym"])
        assert np.array_equal(q.outlier_idx.cpu().numpy().view(np.uint32), base["outlier_idx"])


def test_search_over_bits(ctx):
    rng = np.random.default_rng(15)
    fam = families(rng, 50001)
    xs = [fam["t3"], fam["zeros"], fam["positive"], fam["lattice"], fam["t3"][:7], fam["wide"][:3000]]
    cfgs = [(0, 100000, 1000), (0, 0, 0), (0, 300000, 100), (0, 0, 1000), (0, 0, 0), (0, 50000, 0)]
    for eps in (1e-2, 1e-4, 0.5):
        check_search(ctx, xs, cfgs, eps, 0.01, 0.2, 100, 21)
    # on top of a grid search that holds every width of the fractions in use
    grid = [(b, p, o) for b in range(2, 9) for (p, o) in ((100000, 1000), (0, 0))]
    check_search(ctx, [fam["t3"], fam["zeros"]], [(0, 100000, 1000), (0, 0, 0)], 1e-3, 0.02, 0.4, 50, 22,
                 reuse_grid=grid)


@pytest.mark.parametrize("m", [1, 63, 64, 65, 257, 1023, 1024, 1025, 4096, 4097])
def test_search_over_bits_with_so_many_buckets(ctx, m):
    """Bucket lists at the edges of a wave, of one bucket per thread and of LDS."""
    rng = np.random.default_rng(m)
    gamma = 1.01 / 0.99
    mag = 1e-12 * gamma ** (np.arange(m) // 2 + 0.5)
    x = np.where(np.arange(m) % 2 == 0, mag, -mag)
    x = rng.permutation(np.repeat(x, rng.integers(1, 4, m))).astype(np.float32)
    check_search(ctx, [x, x[:1]], [(0, 0, 0), (0, 0, 0)], 1e-3, 0.01, 0.2, 100, 30 + m)
    base = ref.quantize(x, (8, 0, 0))
    got = sk.quantize_values(x, base["sym"], 256, 0.01, 0.2, rng.uniform(size=256), 1)["n_buckets"]
    assert got == m


def test_stand_alone_state_is_not_offered_for_reuse(ctx):
    """Stand-alone sketch calls search for thresholds and counts only; an equal-frequency quantize
    that asks for the state of the last search must then be refused."""
    from paper_2306_11800_amd import api
    rng = np.random.default_rng(16)
    x = dev((rng.standard_t(3, 30000) * 0.015).astype(np.float32))
    ctx.quantize_sketch([x], [(4, 100000, 1000)], rng.uniform(size=(1, 256)))
    with pytest.raises(api.InshrError) as e:
        ctx.quantize([x], [(4, 100000, 1000)], reuse_search=True)
    assert e.value.code == -5
    q = ctx.quantize([x], [(4, 100000, 1000)])[0]  # stand-alone works as ever
    assert q.n_kept > 0


def test_degenerate_tensors(ctx):
    """All zeros, a constant, one value, zeros with one other value, the ends of the fp32 range; an
    error bound of zero."""
    xs = [np.zeros(5000, np.float32), np.full(20000, -0.37, np.float32), np.array([1e-30], np.float32),
          np.concatenate([np.zeros(100, np.float32), np.full(50, 2.5, np.float32)]),
          np.array([3.0e38, -3.0e38, 1.0, 0.0], np.float32)]
    fractions = [(0, 0, 0), (0, 100000, 1000), (0, 0, 0), (0, 300000, 0), (0, 0, 0)]
    for eps in (1e-2, 0.0):
        check_search(ctx, xs, fractions, eps, 0.01, 0.2, 100, 77)
    check(ctx, xs, [(3, 0, 0), (8, 100000, 1000), (2, 0, 0), (5, 300000, 0), (4, 0, 0)], 0.01, 0.2, 100, 78)


def test_argument_errors(ctx):
    from paper_2306_11800_amd import api
    x = dev(np.ones(100, np.float32))
    uni = np.full((1, 256), 0.5)
    for kw in (dict(alpha=0.001), dict(alpha=0.7), dict(sigma=1.5), dict(sigma=-0.1)):
        with pytest.raises(api.InshrError) as e:
            ctx.quantize_sketch([x], [(4, 0, 0)], uni, **kw)
        assert e.value.code == -2
    with pytest.raises(api.InshrError) as e:
        ctx.quantize_sketch([x], [(4, 0, 0)], np.full((1, 256), 1.0))
    assert e.value.code == -1


def test_restore_round_trip(ctx):
    rng = np.random.default_rng(13)
    x = (rng.standard_t(3, 40000) * 0.015).astype(np.float32)
    uni = rng.uniform(size=(1, 256))
    qs, _ = ctx.quantize_sketch([dev(x)], [(4, 100000, 1000)], uni)
    y = ctx.dequantize(qs)[0].cpu().numpy()
    q = qs[0]
    sym = ref.unpack(q.packed.cpu().numpy().view(np.uint64), x.size, 5)
    cb = q.codebook.cpu().numpy()
    want = np.where(sym == 0, np.float32(0), np.where(sym == 1, x, cb[np.maximum(sym.astype(np.int64) - 2, 0)]))
    assert np.array_equal(y.view(np.uint32), want.astype(np.float32).view(np.uint32))
    # every quantized value decodes to the nearest centre
    m = sym >= 2
    d = np.abs(x[m].astype(np.float64)[:, None] - cb[:16].astype(np.float64)[None, :])
    assert np.all(np.abs(y[m].astype(np.float64) - x[m]) <= d.min(axis=1) * (1 + 1e-12))


def test_sketch_quantile_estimates_equal_the_oracle(ctx):
    """Sec. 4.3: the sketch as the quantile estimator, on its own: the bucket that holds the rank is
    an integer decision, so the estimates equal the oracle's to the last bit; and they lie within
    alpha of numpy's order statistic."""
    rng = np.random.default_rng(140)
    qs = [0.0, 0.05, 0.1, 0.2, 0.4, 0.5, 0.9, 0.999, 0.9999, 1.0]
    xs = [(0.02 * rng.standard_t(4, n)).astype(np.float32) for n in (1, 7, 65_536, 65_537, 300_001)]
    xs[2][::3] = 0.0
    xs[3][:100] = np.float32(1e-41)           # denormals
    xs.append(np.zeros(1000, np.float32))
    for alpha in (0.01, 0.05):
        got = ctx.sketch_quantiles([dev(x) for x in xs], qs, alpha)
        for x, row in zip(xs, got):
            mag = np.sort(np.abs(x))
            for q, est in zip(qs, row):
                assert est == sk.quantile_estimate(np.abs(x), q, alpha), (x.size, q, alpha)
                exact = float(mag[int(np.floor(q * (x.size - 1)))])
                assert abs(est - exact) <= alpha * exact * (1 + 1e-6)
    # a tensor that does not start at a 16-byte boundary
    t = dev(xs[4])
    got = ctx.sketch_quantiles([t[1:]], qs, 0.01)[0]
    assert got == [sk.quantile_estimate(np.abs(xs[4][1:]), q, 0.01) for q in qs]
    from paper_2306_11800_amd import api
    bad = xs[1].copy()
    bad[3] = np.nan
    with pytest.raises(api.InshrError) as e:
        ctx.sketch_quantiles([dev(bad)], [0.5], 0.01)
    assert e.value.code == -3
    with pytest.raises(api.InshrError):
        ctx.sketch_quantiles([dev(xs[1])], [1.5], 0.01)


def test_search_over_pairs_and_bits(ctx):
    """Sec. 5 with the bins of Algorithm 2 over (prune, protect) pairs as well as the bit width: every
    row of the table against the oracle's search over the bits for that pair, the winner against the
    oracle's rule (least payload within the bound, else the least 8-bit error), and the winner's codes
    against the oracle's quantizer."""
    rng = np.random.default_rng(150)
    fam = families(rng, 30001)
    xs = [fam["t3"], fam["zeros"], fam["positive"][:5000], fam["t3"][:9]]
    pairs = [(0, 0), (100000, 0), (100000, 1000), (300000, 1000), (500000, 10000)]
    uni = rng.uniform(size=(len(xs), 256))
    for eps in (1e-2, 2e-4, 1e-9):
        qs, best, rows, table = ctx.search_sketch_grid([dev(x) for x in xs], pairs, uni, eps, alpha=0.01, sigma=0.2)
        for i, x in enumerate(xs):
            bases = [ref.quantize(x, (8, p, o)) for p, o in pairs]
            classes = [np.minimum(b["sym"], 2) for b in bases]
            want = sk.search_grid(x, classes, 0.01, 0.2, uni[i], 100, eps)
            border = False
            for q in range(len(pairs)):
                r, ch = want["per_pair"][q], table[i][q]
                for b in range(2, 9):
                    assert abs(ch["sse"][b - 2] - r["sse"][b]) <= 1e-6 * r["sse"][b] + 1e-12 * r["sumsq"]
                    if r["sumsq"] > 0 and abs(r["sse"][b] / r["sumsq"] - eps) <= 4e-6 * eps:
                        border = True
                if not border:
                    assert (ch["best_bits"], ch["feasible"]) == (r["best_bits"], r["feasible"])
            if border:
                continue
            # (an 8-bit error that ties between pairs to the last digits may fall either way)
            if not want["feasible"]:
                e8 = sorted(want["per_pair"][q]["sse"][8] for q in range(len(pairs)))
                if len(e8) > 1 and e8[1] - e8[0] <= 1e-6 * e8[0] + 1e-12 * want["per_pair"][0]["sumsq"]:
                    continue
            assert (best[i], rows[i]["best_bits"], rows[i]["feasible"]) == (want["pair"], want["bits"], want["feasible"]), (i, eps)
            run = want["per_pair"][want["pair"]]["runs"][want["bits"]]
            got = ref.unpack(qs[i].packed.cpu().numpy().view(np.uint64), x.size, want["bits"] + 1)
            assert np.array_equal(got, run["sym"])
            np.testing.assert_allclose(qs[i].codebook.cpu().numpy(), run["codebook"], rtol=1e-6, atol=0)
            assert np.array_equal(qs[i].outlier_idx.cpu().numpy().view(np.uint32), bases[want["pair"]]["outlier_idx"])
