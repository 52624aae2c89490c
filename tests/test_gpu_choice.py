"""A search that is asked for its choice alone (want_scores=False) against one that scores every
configuration: the choice, and what the quantizer gives afterwards for the chosen configuration and for
others of the grid, on value families at sizes that the sweeps search, at bounds that leave the choice
open, that all and that no configuration meets."""
import numpy as np
import pytest
import torch

from oracle import ref
from paper_2306_11800_amd import api, synth
from test_gpu_full_size import unpack
from test_gpu_fuzz import family
from test_gpu_parity import check_quantized
from test_gpu_small import KINDS, repeated

pytestmark = pytest.mark.gpu

GRIDS = {
    "full": synth.grid_full(),
    "bins": synth.grid_paper(prune=(0.0, 0.2, 0.5), protect=(0.0, 0.005, 0.02), bins=(2, 3, 4, 6, 12, 16, 256)),
}


def dev(x):
    return torch.from_numpy(x).to("cuda:0")


def same(a, b):
    """Integers equal, centres to 1e-6 (their sums are grouped by other edge lists)."""
    assert len(a) == len(b)
    for x, y in zip(a, b):
        assert (x.n_pruned, x.n_outlier, x.n_kept, x.K) == (y.n_pruned, y.n_outlier, y.n_kept, y.K)
        assert torch.equal(x.packed, y.packed)
        assert torch.equal(x.boundaries[:x.K - 1].view(torch.int32), y.boundaries[:y.K - 1].view(torch.int32))
        assert torch.equal(x.outlier_idx[:x.n_outlier], y.outlier_idx[:y.n_outlier])
        assert torch.equal(x.outlier_val[:x.n_outlier], y.outlier_val[:y.n_outlier])
        np.testing.assert_allclose(x.codebook[:x.K].cpu().numpy(), y.codebook[:y.K].cpu().numpy(), rtol=1e-6)


@pytest.mark.parametrize("ordered", [True, False])
@pytest.mark.parametrize("grid", sorted(GRIDS))
def test_choice_alone(monkeypatch, grid, ordered):
    monkeypatch.setenv("INSHR_NO_LDS_ORDER", "0" if ordered else "1")
    scored, bare = api.Context(torch.device("cuda:0")), api.Context(torch.device("cuda:0"))
    g = GRIDS[grid]
    rng = np.random.default_rng(41)
    sizes = [16385, 40_000, 131_073, 700_001] if ordered else [16385, 70_000]
    xs = [family(rng, k, n) for k in range(10) for n in sizes] + [repeated(rng, k, n) for k in KINDS for n in sizes[:2]]
    ts = [dev(x) for x in xs] + [dev(family(rng, 0, 300))]  # (and one that a workgroup searches by itself)
    _, _, sc = scored.search(ts, g, synth.EPS_DEFAULT)
    rel = np.array([s.sse / s.sumsq if s.sumsq else 0.0 for s in sc]).reshape(len(ts), len(g))
    # 2e-9: below what the sums resolve; the middle configuration's own error: open for its tensor
    for eps in [synth.EPS_DEFAULT, 1.0, 2e-9, float(np.sort(rel[0])[len(g) // 2]), float(np.sort(rel[7])[len(g) // 4])]:
        want = scored.search(ts, g, eps)
        got = bare.search(ts, g, eps, want_scores=False)
        near = np.abs(rel - eps) <= 4e-6 * eps + 1e-12  # (an error that rounds to the bound may fall on either side)
        for t in range(len(ts)):
            if not near[t].any() and eps > 1e-8:
                assert (got[0][t], got[1][t]) == (want[0][t], want[1][t]), (t, eps)
        for cfgs in ([g[b] for b in want[0]], [g[(7 * t + 3) % len(g)] for t in range(len(ts))]):
            same(bare.quantize(ts, cfgs, reuse_search=True), scored.quantize(ts, cfgs, reuse_search=True))
    scored.close()
    bare.close()


def choose(ctx, ts, g, eps, groups=None):
    """A search for its choice alone, and which means it took for what the bounds leave open: one configuration's error by
    the quantizer's sweep ("one"), one configuration or all of them by the scored search's kernels ("grid")."""
    ctx.profile(True)
    best, feasible, _ = ctx.search(ts, g, float(eps), want_scores=False, groups=groups)
    kernels = ctx.profile_read()
    ctx.profile(False)
    return (list(best), list(feasible)), {m for m, k in (("one", "k_fuse_dry"), ("grid", "k_final")) if k in kernels}


def check_choice(scored, bare, ts, g, eps, means):
    best, feasible, _ = scored.search(ts, g, float(eps))
    got, took = choose(bare, ts, g, eps)
    assert got == (list(best), list(feasible)) and took == means, (eps, got, took)
    n = len(g)
    for cfgs in ([g[b] for b in best], [g[(b + n // 2) % n] for b in best]):
        same(bare.quantize(ts, cfgs, reuse_search=True), scored.quantize(ts, cfgs, reuse_search=True))


@pytest.fixture
def two_contexts():
    pair = [api.Context(torch.device("cuda:0")) for _ in range(2)]
    yield pair
    for c in pair:
        c.close()


AROUND = (1 - 2e-4, 1 + 2e-4)  # of an error: closer than the bounds are, farther than rounding


@pytest.mark.parametrize("n", [16_385, 300_001, 2_500_000])
def test_choice_that_hangs_on_one_configuration(two_contexts, n):
    """A bound just above and just below the error of a configuration that costs less than all more accurate ones: its
    error alone is worked out, by the quantizer's sweep.  Among them the most accurate of all, with none to fall back on."""
    g = GRIDS["full"]
    x = dev(family(np.random.default_rng(47), 0, n))
    scored, bare = two_contexts
    _, _, sc = scored.search([x], g, synth.EPS_DEFAULT)
    order = sorted(range(len(g)), key=lambda k: sc[k].sse)
    hang = [k for i, k in enumerate(order) if all(sc[k].cost_bits < sc[j].cost_bits for j in order[:i])]
    assert hang[0] == order[0] and len(hang) >= 8
    for k in hang[::3]:
        for f in AROUND:
            check_choice(scored, bare, [x], g, sc[k].sse / sc[k].sumsq * f, {"one"})


def test_choice_that_hangs_with_shared_thresholds(two_contexts):
    """The same for tensors whose thresholds are their group's."""
    rng = np.random.default_rng(52)
    ts, groups = [dev(family(rng, 0, n)) for n in (300_001, 90_000, 120_001)], [0, 1, 0]
    g = [(4, 100_000, 0), (8, 100_000, 0)]
    scored, bare = two_contexts
    _, _, sc = scored.search(ts, g, synth.EPS_DEFAULT, groups=groups)
    for t in range(3):
        for f in AROUND:
            eps = sc[t * len(g)].sse / sc[t * len(g)].sumsq * f
            best, feasible, _ = scored.search(ts, g, float(eps), groups=groups)
            got, took = choose(bare, ts, g, eps, groups)
            assert got == (list(best), list(feasible)) and "one" in took, (t, eps, took)


def crowded(rng, n):
    """A quarter of the values is one number: a bin that a boundary lies in holds more than one wave of the sweep reads."""
    y = family(rng, 0, n)
    y[rng.random(n) < 0.25] = np.float32(0.01)
    return y


@pytest.mark.parametrize("kind,cheap,means", [("long lists", (4, 0, 20_000), {"grid"}), ("crowded bin", (4, 0, 1000), {"one", "grid"}),
                                              ("crowded bin", (4, 0, 0), {"one", "grid"})])
def test_choice_that_hangs_on_what_the_sweep_does_not_hold(two_contexts, kind, cheap, means):
    """More protected values than its lists are made for: not tried.  A bin too full for it: tried, and left to the others."""
    rng = np.random.default_rng(48)
    g = [cheap, (8, 0, cheap[2])]
    x = dev(family(rng, 0, 300_001) if kind == "long lists" else crowded(rng, 400_001))
    scored, bare = two_contexts
    _, _, sc = scored.search([x], g, synth.EPS_DEFAULT)
    for ts in ([x], [x, dev(family(rng, 0, 90_000)), 2 * x]):
        for f in AROUND:
            check_choice(scored, bare, ts, g, sc[0].sse / sc[0].sumsq * f, means)


def with_tail(ctx, rng, n, g, k, rel):
    """Values whose relative error with configuration k is rel: a twentieth of them as much larger as it takes."""
    x = dev(rng.standard_normal(n).astype(np.float32))
    some = torch.from_numpy(rng.random(n) < 0.05).to("cuda:0")
    lo, hi = 0.1, 100.0
    for _ in range(40):
        s = (lo * hi) ** 0.5
        y = torch.where(some, x * s, x)
        _, _, sc = ctx.search([y], g, synth.EPS_DEFAULT)
        r = sc[k].sse / sc[k].sumsq
        if abs(r / rel - 1) < 5e-5:
            return y
        lo, hi = (s, hi) if r < rel else (lo, s)
    raise AssertionError((r, rel, s))


def test_choices_of_one_call_that_hang_on_different_means(two_contexts):
    """At one bound: a tensor that the sweep holds, one with a bin too full for it, one that is settled by its bounds, a small
    one; and a tensor with one configuration open beside one with two (equal errors: a protect fraction that protects none
    of its values), whose whole grid is scored, which the first one's configuration then joins."""
    rng = np.random.default_rng(49)
    scored, bare = two_contexts
    g = [(4, 0, 1000), (8, 0, 1000)]
    bad = dev(crowded(rng, 400_001))
    _, _, sc = scored.search([bad], g, synth.EPS_DEFAULT)
    rel = sc[0].sse / sc[0].sumsq
    held = with_tail(scored, rng, 300_001, g, 0, rel)
    ts = [dev(family(rng, 0, 50_000)), held, dev(family(rng, 0, 700)), bad, 4 * held, 4 * bad]
    for f in (1 - 4e-4, 1 + 4e-4):
        check_choice(scored, bare, [held], g, rel * f, {"one"})
        check_choice(scored, bare, ts, g, rel * f, {"one", "grid"})
    g = [(4, 0, 0), (4, 0, 2), (8, 0, 0)]
    one = (rng.standard_normal(2_500_000) * np.where(rng.random(2_500_000) < 0.01, 3.0, 1.0)).astype(np.float32)
    one[1_000_003] = one[77] = 300.0
    one = dev(one)
    _, _, sc = scored.search([one], g, synth.EPS_DEFAULT)
    rel = sc[1].sse / sc[1].sumsq
    assert sc[0].sse > 1.1 * sc[1].sse
    two = with_tail(scored, rng, 300_001, g, 1, rel)
    for f in (1 - 4e-4, 1 + 4e-4):
        check_choice(scored, bare, [one], g, rel * f, {"one"})
        check_choice(scored, bare, [two], g, rel * f, {"grid"})
        check_choice(scored, bare, [one, two], g, rel * f, {"grid"})


def test_shares_of_the_pool_grow_in_the_quantizer(monkeypatch):
    """One value makes up most of the tensor and holds boundaries: all its keys are gathered."""
    rng = np.random.default_rng(42)
    x = repeated(rng, "run", 400_000)
    y = np.where(rng.random(400_000) < 0.8, np.float32(0.25), x).astype(np.float32)
    ts = [dev(y), dev(family(rng, 0, 50_000))]
    want = api.Context(torch.device("cuda:0"))
    b, _, _ = want.search(ts, GRIDS["full"], 0.01)
    monkeypatch.setenv("INSHR_POOL_WCAP", "1")
    small = api.Context(torch.device("cuda:0"))
    b2, _, _ = small.search(ts, GRIDS["full"], 0.01, want_scores=False)
    assert list(b) == list(b2)
    cfgs = [GRIDS["full"][k] for k in b]
    same(small.quantize(ts, cfgs, reuse_search=True), want.quantize(ts, cfgs, reuse_search=True))
    same(small.quantize(ts, cfgs), want.quantize(ts, cfgs, reuse_search=True))
    want.close()
    small.close()


def test_pooled_choice_and_sketch_on_top(monkeypatch):
    """Thresholds per group without scores; the sketch quantizer reuses a search that only chose."""
    rng = np.random.default_rng(43)
    ts = [dev(family(rng, k, n)) for k, n in [(0, 90_000), (0, 30_001), (9, 50_000), (9, 900)]]
    ctx, bare = api.Context(torch.device("cuda:0")), api.Context(torch.device("cuda:0"))
    groups = [0, 0, 1, 1]
    want = ctx.search(ts, GRIDS["full"], 0.01, groups=groups)
    got = bare.search(ts, GRIDS["full"], 0.01, want_scores=False, groups=groups)
    assert list(want[0]) == list(got[0]) and list(want[1]) == list(got[1])
    # (a member's share of the protected values is not bounded by the fraction: a configuration without any)
    cfg = [(4, 200_000, 0)] * len(ts)
    same(bare.quantize(ts, cfg, reuse_search=True), ctx.quantize(ts, cfg, reuse_search=True))
    u = rng.uniform(size=(len(ts), 256))
    cfgs = [(8, 200_000, 1000)] * len(ts)
    a = ctx.search(ts, GRIDS["full"], 0.01) and ctx.search_sketch(ts, cfgs, u, 0.01, reuse_search=True)
    b = bare.search(ts, GRIDS["full"], 0.01, want_scores=False) and bare.search_sketch(ts, cfgs, u, 0.01, reuse_search=True)
    same(a[0], b[0])
    np.testing.assert_allclose([c["sse"] for c in a[1]], [c["sse"] for c in b[1]], rtol=1e-6, atol=1e-12)
    ctx.close()
    bare.close()


@pytest.mark.parametrize("off", [1, 2, 3])
def test_slices_that_start_anywhere(off):
    """16-byte loads from tensors that are aligned to 4 bytes only: the same as from aligned copies."""
    rng = np.random.default_rng(44)
    sizes = [16_384 + off, 24_576, 90_000 + off]  # (a tile of the sweeps is a multiple of 4096)
    flat = dev(family(rng, 1, 262_144))
    cuts = [flat[k * 65_536 + off:][:n] for k, n in enumerate(sizes)]
    assert all(t.data_ptr() % 16 == 4 * off for t in cuts)
    copies = [t.clone() for t in cuts]
    a, b = api.Context(torch.device("cuda:0")), api.Context(torch.device("cuda:0"))
    for want_scores in (True, False):
        ra, rb = (c.search(ts, GRIDS["full"], 0.01, want_scores=want_scores) for c, ts in ((a, cuts), (b, copies)))
        assert list(ra[0]) == list(rb[0]) and list(ra[1]) == list(rb[1])
        cfgs = [GRIDS["full"][k] for k in ra[0]]
        same(a.quantize(cuts, cfgs, reuse_search=True), b.quantize(copies, cfgs, reuse_search=True))
    u = rng.uniform(size=(len(cuts), 256))
    cfgs = [(8, 200_000, 1000)] * len(cuts)
    same(a.search_sketch(cuts, cfgs, u, 0.01)[0], b.search_sketch(copies, cfgs, u, 0.01)[0])
    a.close()
    b.close()


def test_more_tensors_than_a_grid_dimension():
    """More tensors for the sweeps than the second and third dimension of a grid hold (65535), one call with one
    configuration: every tensor is quantized as by itself."""
    n, n_t, kinds, cfg = 16_385, 65_540, 64, (4, 200_000, 1000)
    flat = dev(family(np.random.default_rng(45), 1, n + kinds))
    ctx = api.Context(torch.device("cuda:0"))
    want = [ctx.quantize([flat[k:k + n]], [cfg])[0] for k in range(kinds)]
    rows = dict(packed=(-(-n * api.symbol_bits(16) // 64), torch.int64), codebook=(256, torch.float32),
                boundaries=(255, torch.float32), outlier_idx=(n // 1000 + 1, torch.int32),
                outlier_val=(n // 1000 + 1, torch.float32))
    bufs = {k: torch.zeros(n_t, w, dtype=t, device="cuda:0") for k, (w, t) in rows.items()}
    out = [api.Quantized(n, 4, b) for b in zip(*(b.unbind(0) for b in bufs.values()))]
    cuts = [flat[k:k + n] for k in range(kinds)]
    got = ctx.quantize([cuts[t % kinds] for t in range(n_t)], [cfg] * n_t, out=out)
    assert len({(q.n_pruned, q.n_outlier, q.n_kept) for q in got[::kinds]}) == 1
    for k, w in enumerate(want):
        assert (got[k].n_pruned, got[k].n_outlier, got[k].n_kept) == (w.n_pruned, w.n_outlier, w.n_kept)
        for name in rows:
            x = getattr(w, name)
            part = bufs[name][k::kinds, :x.numel()]
            if name == "codebook":  # (its sums are exact integers: equal too)
                assert torch.equal(part, x.expand_as(part)), k
            else:
                assert torch.equal(part.view(torch.int32), x.view(torch.int32).expand(part.shape[0], -1)), (name, k)
    ctx.close()


def test_quantizing_again_from_a_choice():
    """What the sweep worked out stays in the state: a further call for the same configuration gives the same bytes
    without it (k_quant), also after calls for others; protected values nowhere, everywhere, and in some tiles only."""
    rng = np.random.default_rng(46)
    n = 150_001
    some = family(rng, 0, n)
    some[40_000:41_000] *= np.float32(50)
    xs = [some, family(rng, 0, 16_385), family(rng, 1, n), np.zeros(n, np.float32)]
    ts = [dev(x) for x in xs]
    ctx, want = api.Context(torch.device("cuda:0")), api.Context(torch.device("cuda:0"))
    g = GRIDS["full"]
    best = ctx.search(ts, g, 0.01, want_scores=False)[0]
    want.search(ts, g, 0.01)
    first, other, bare = [g[b] for b in best], [(3, 50_000, 1000)] * len(ts), [(8, 0, 0)] * len(ts)
    for cfgs in (first, other, bare):
        a = ctx.quantize(ts, cfgs, reuse_search=True)
        ctx.profile(True)
        b = ctx.quantize(ts, cfgs, reuse_search=True)
        kernels = ctx.profile_read()
        ctx.profile(False)
        assert "k_fuse" not in kernels and "k_quant" in kernels, kernels
        same(a, b)
        for x, y in zip(a, b):
            assert torch.equal(x.codebook, y.codebook)
        same(b, want.quantize(ts, cfgs, reuse_search=True))
    same(ctx.quantize(ts, first, reuse_search=True), want.quantize(ts, first, reuse_search=True))
    ctx.close()
    want.close()


@pytest.mark.parametrize("bits", range(1, 9))
def test_symbols_of_every_width(bits):
    """Both sweeps pack 2 to 9 bits a symbol, wave by wave: ends inside a wave's words, units of one tile and (70 M values
    on 256 workgroups) of more than the 16 whose symbols are found by cells, with protected values in every tile, in one
    and in none.  Every whole number as the oracle's, or as the thresholds and boundaries say."""
    rng = np.random.default_rng(49)
    ctx = api.Context(torch.device("cuda:0"))
    for n in (16_385, 49_229, 330_001):
        x = (0.02 * rng.standard_t(4, n)).astype(np.float32)
        x[20_000:20_900] *= np.float32(40 if n > 330_000 else 1)
        for cfg in ((bits, 200_000, 1000), (bits, 200_000, 0)):
            t = [dev(x)]
            ctx.search(t, [cfg], synth.EPS_DEFAULT, want_scores=False)
            q = ctx.quantize(t, [cfg], reuse_search=True)
            check_quantized(q[0], x, cfg)
            ctx.profile(True)
            again = ctx.quantize(t, [cfg], reuse_search=True)
            assert "k_quant" in ctx.profile_read()
            ctx.profile(False)
            same(again, q)
    n, cfg = 70_000_037, (bits, 200_000, 1000)
    x = torch.empty(n, device="cuda:0")
    x.normal_(generator=torch.Generator(device="cuda:0").manual_seed(50))
    first = ctx.quantize([x], [cfg])
    again = ctx.quantize([x], [cfg], reuse_search=True)
    same(again, first)
    q = again[0]
    sym = torch.bucketize(x, q.boundaries[:q.K - 1].contiguous(), right=True) + 2
    sym[x.abs() < q.tau_prune] = 0
    sym[x.abs() > q.tau_outlier] = 1
    assert torch.equal(unpack(q.packed, n, bits + 1).long(), sym)
    assert torch.equal(q.outlier_idx[:q.n_outlier].long(), (sym == 1).nonzero()[:, 0])
    assert torch.equal(q.outlier_val[:q.n_outlier], x[sym == 1])
    ctx.close()


@pytest.mark.parametrize("levels", [0, 4000, 300, 40])
@pytest.mark.parametrize("n", [16_385, 120_001])
def test_values_in_bins_with_breakpoints(levels, n):
    """Values whose symbol the sweep works out one by one, from a few of a wave's 256 to all of them: the fewer distinct values
    there are, the more share a bin with a boundary (40 levels: nearly every bin that holds any).  Also with half of the
    values zero and boundaries there.  Against the oracle."""
    rng = np.random.default_rng(51)
    ctx = api.Context(torch.device("cuda:0"))
    x = rng.standard_normal(n).astype(np.float32)
    if levels:
        x = np.round(x * np.float32(levels / 8)) / np.float32(levels / 8)
    half = x.copy()
    half[rng.random(n) < 0.5] = 0.0
    half[::7] *= np.float32(-1)  # (zeros of both signs)
    for y in (x, half):
        for cfg in ((8, 200_000, 1000), (5, 0, 5000), (2, 0, 0)):
            ctx.profile(True)
            q = ctx.quantize([dev(y)], [cfg])
            kernels = ctx.profile_read()
            ctx.profile(False)
            assert "k_fuse" in kernels, kernels
            check_quantized(q[0], y, cfg)
    ctx.close()


def test_tensors_of_every_kind_in_one_call():
    """One call with tensors that the state holds, that the sweep takes, that it gives up (one bin holds more values
    than a wave should read), that protect too much for its lists, and a small one: several passes, each on its own
    tensors only."""
    rng = np.random.default_rng(47)
    n = 200_001
    crowd = family(rng, 0, n)
    crowd[:140_000] = np.float32(0.25)
    ts = [dev(x) for x in (family(rng, 0, n), family(rng, 1, n), crowd, family(rng, 2, n), family(rng, 0, 900))]
    ctx, want = api.Context(torch.device("cuda:0")), api.Context(torch.device("cuda:0"))
    g = GRIDS["bins"]
    few, many = (0, 200_000, 5000, 16), (0, 200_000, 20_000, 16)
    want.search(ts, g, 0.01)
    ctx.search(ts, g, 0.01, want_scores=False)
    ctx.quantize(ts, [few, many, many, many, few], reuse_search=True)  # (the first stays in the state)
    cfgs = [few, few, few, (0, 0, 20_000, 16), few]
    for again in (False, True):
        ctx.profile(True)
        got = ctx.quantize(ts, cfgs, reuse_search=True)
        kernels = ctx.profile_read()
        ctx.profile(False)
        same(got, want.quantize(ts, cfgs, reuse_search=True))
        assert ("k_fuse" in kernels, "k_gather" in kernels) == (not again, not again), kernels
        assert kernels["k_quant"][1] == (1 if again else 2), kernels
    ctx.close()
    want.close()


def test_sums_of_long_units(monkeypatch):
    """Units of more than 64 tiles (the sweep empties its cells after as many): one tensor of 131 M values three
    times in one call on 256 workgroups gives what it gives alone in units of 16 tiles, and its centres are
    the means of the values of their bins."""
    n, cfg = 131_072_000 + 5, (5, 200_000, 1000)
    x = torch.empty(n, device="cuda:0")
    x.normal_(generator=torch.Generator(device="cuda:0").manual_seed(48))
    alone = api.Context(torch.device("cuda:0"))
    want = alone.quantize([x], [cfg])[0]
    monkeypatch.setenv("INSHR_WG_PER_CU", "1")
    ctx = api.Context(torch.device("cuda:0"))
    ctx.profile(True)
    got = ctx.quantize([x] * 3, [cfg] * 3)
    kernels = ctx.profile_read()
    assert "k_fuse" in kernels and "k_quant" not in kernels, kernels
    for q in got:
        same([q], [want])
        assert torch.equal(q.codebook, want.codebook)  # (the sums are exact integers)
    ctx.close()
    alone.close()
    kept = x[(x.abs() >= want.tau_prune) & (x.abs() <= want.tau_outlier)]
    assert kept.numel() == want.n_kept
    b = torch.bucketize(kept, want.boundaries[:31], right=True)
    s = torch.zeros(32, dtype=torch.float64, device="cuda:0").index_add_(0, b, kept.double())
    mean = s / torch.bincount(b, minlength=32)
    # (2^-24 of rounding to fp32; the fp64 sums of 3 M values of one sign are exact to 1e-9)
    np.testing.assert_allclose(want.codebook[:32].cpu().numpy(), mean.cpu().numpy(), rtol=1e-7)


@pytest.mark.parametrize("values", ["protected", "open"])
def test_lists_that_overflow(values):
    """Values of one wave's list that lie side by side, more than its share takes: protected ones (the largest
    percent of the tensor in one run), and values of one bin that holds boundaries.  The tensor is given up by
    the sweep and goes through k_gather and k_quant; the one beside it does not."""
    rng = np.random.default_rng(49)
    n = 1 << 20
    x, beside = family(rng, 0, n), family(rng, 0, n)
    if values == "protected":
        x[100_000:110_485] = np.float32(50) * (1 + rng.random(10_485).astype(np.float32))
    else:
        x[100_000:130_000] = np.float32(np.median(np.abs(x)))
    cfg, g = (8, 0, 10_000), [(8, 0, 10_000)]
    ts = [dev(x), dev(beside)]
    ctx = api.Context(torch.device("cuda:0"))
    ctx.search(ts, g, 0.01, want_scores=False)
    ctx.profile(True)
    got = ctx.quantize(ts, [cfg] * 2, reuse_search=True)
    kernels = ctx.profile_read()
    ctx.profile(False)
    assert "k_fuse" in kernels and kernels["k_gather"][1] == kernels["k_quant"][1] == 1, kernels
    same(got, ctx.quantize(ts, [cfg] * 2))
    for q, v in zip(got, (x, beside)):
        r = ref.quantize(v, cfg)
        assert np.array_equal(q.packed.cpu().numpy().view(np.uint64), ref.pack(r["sym"], 9))
        np.testing.assert_allclose(q.codebook.cpu().numpy(), r["codebook"], rtol=1e-6)
        assert np.array_equal(q.outlier_idx.cpu().numpy()[:q.n_outlier], np.flatnonzero(r["sym"] == 1))
    ctx.close()


@pytest.mark.parametrize("values", ["heavy", "few", "run", "family 0", "family 1"])
def test_bounds_that_sit_on_an_error(values):
    """eps just beside the exact error of a configuration: the choice is the scored search's, also where one value
    makes up nearly all of a tensor and the boundaries lie among few others."""
    rng = np.random.default_rng(50)
    n = 300_001 if values.startswith("family") else 17_001  # (the scored search is slow where a bin holds most values)
    if values == "heavy":
        x = np.full(n, np.float32(0.95))
        x[:n // 100] = np.exp(rng.normal(3, 0.5, n // 100)).astype(np.float32)
        x = rng.permutation(x)
    elif values == "few":
        x = rng.choice(np.array([-1.5, -0.1, 0.0, 0.3, 0.30001, 0.31, 2.0, 7.0], np.float32), n)
    else:
        x = repeated(rng, "run", n) if values == "run" else family(rng, int(values[-1]), n)
    ts, g = [dev(x)], GRIDS["full"]
    scored, bare = api.Context(torch.device("cuda:0")), api.Context(torch.device("cuda:0"))
    rel = np.array([s.sse / s.sumsq for s in scored.search(ts, g, 0.01)[2]])
    for k in range(4, len(g), 9):
        for f in (1 - 1e-4, 1 - 2e-5, 1 + 2e-5, 1 + 1e-4):
            eps = float(rel[k] * f)
            if (np.abs(rel - eps) <= 4e-6 * eps + 1e-12).any():
                continue  # (an error that rounds to the bound may fall on either side)
            want, got = scored.search(ts, g, eps), bare.search(ts, g, eps, want_scores=False)
            assert (got[0][0], got[1][0]) == (want[0][0], want[1][0]), (k, f)
    scored.close()
    bare.close()
