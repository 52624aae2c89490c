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
