"""What a call uploads and clears, by numbers of tensors at which its parts end inside and at the ends of the pieces and
workgroups that copy them: every tensor of a call comes out as in a call by itself."""
import numpy as np
import pytest
import torch

from paper_2306_11800_amd import api, synth

pytestmark = pytest.mark.gpu
SIZES = (300, 5_000, 16_385, 40_000)  # (by one workgroup each, by the sweeps)


def step(ctx, ts, prev):
    grid = synth.grid_small()
    best, feasible, _ = ctx.search(ts, grid, 0.01, want_scores=False)
    q = ctx.quantize(ts, [grid[b] for b in best], reuse_search=True)
    d = ctx.delta(prev, q)
    words = ctx.reconstruct(prev, d, [x.bits for x in q], [x.K for x in q])
    out = [torch.empty_like(t) for t in ts]
    ctx.dequantize(q, out=out)
    ctx.sync()
    return [(best[i], feasible[i], q[i].packed, d[i].packed[:(d[i].n * d[i].delta_bits + 63) // 64], words[i], out[i])
            for i in range(len(ts))]


@pytest.mark.parametrize("n_t", [1, 2, 63, 127, 128, 129, 146, 147, 300, 1171])
def test_calls_on_many_tensors(n_t):
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(3)
    kinds = [torch.empty(n, device="cuda:0").normal_(0, 0.02, generator=gen) for n in SIZES]
    ctx = api.Context(torch.device("cuda:0"))
    prev = ctx.quantize(kinds, [(4, 200_000, 1000)] * len(kinds))
    want = [step(api.Context(torch.device("cuda:0")), [t], [p])[0] for t, p in zip(kinds, prev)]
    rng = np.random.default_rng(n_t)
    for _ in range(2):  # (again in the buffers that the first call left behind, in another order)
        pick = rng.integers(0, len(kinds), n_t)
        got = step(ctx, [kinds[k] for k in pick], [prev[k] for k in pick])
        for k, g in zip(pick, got):
            assert g[:2] == want[k][:2]
            assert all(torch.equal(a, b) for a, b in zip(g[2:5], want[k][2:5]))
            # (centres: sums grouped by other edge lists)
            np.testing.assert_allclose(g[5].cpu().numpy(), want[k][5].cpu().numpy(), rtol=1e-6)
    ctx.close()


@pytest.mark.parametrize("after", ["quantize", "quantize_sketch", "sketch_quantiles", "delta", "reconstruct", "dequantize"])
def test_buffers_that_grow_behind_an_unfinished_delta(after):
    """A delta call returns before its kernels have run.  The call after it wants larger staging buffers and scratch than
    there are: they are exchanged only when nothing reads the old ones any more."""
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(4)
    small = [torch.empty(5_000, device="cuda:0").normal_(0, 0.02, generator=gen) for _ in range(600)]
    ts = [torch.empty(100_000_001, device="cuda:0").normal_(0, 0.02, generator=gen)] + small
    cfg = (4, 200_000, 1000)
    maker = api.Context(torch.device("cuda:0"))
    prev = maker.quantize(ts, [cfg] * len(ts))
    cur = maker.quantize([t * 1.01 for t in ts], [cfg] * len(ts))
    more = maker.quantize(small * 4, [cfg] * (4 * len(small)))
    more_d = maker.delta(more, more)
    want = maker.delta(prev, cur)
    maker.sync()
    for wait in (True, False):
        ctx = api.Context(torch.device("cuda:0"))
        if after == "quantize_sketch":
            ctx.search(ts, [cfg], 0.01, want_scores=False)
        got = ctx.delta(prev, cur)
        if wait:
            ctx.sync()
        if after == "quantize":
            out = [q.packed for q in ctx.quantize(small * 4, [cfg] * (4 * len(small)))]
        elif after == "quantize_sketch":
            u = np.random.default_rng(5).uniform(size=(len(ts), 256))
            out = [q.packed for q in ctx.quantize_sketch(ts, [cfg] * len(ts), u, reuse_search=True)[0]]
        elif after == "sketch_quantiles":
            out = [torch.from_numpy(np.asarray(ctx.sketch_quantiles(ts, [0.1, 0.9])))]
        elif after == "delta":
            out = [d.packed for d in ctx.delta(more, more)]
        elif after == "reconstruct":
            out = ctx.reconstruct(more, more_d, [q.bits for q in more], [q.K for q in more])
        else:
            out = ctx.dequantize(more)
        ctx.sync()
        assert all(torch.equal(a.packed, b.packed) for a, b in zip(got, want))
        if wait:
            first = out
        else:
            assert all(torch.equal(a, b) for a, b in zip(out, first))
        ctx.close()
    maker.close()
