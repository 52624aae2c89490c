"""Tensors that one workgroup searches and quantizes by itself, at the edges of its two size classes
and of a tile, next to tensors that the sweeps search, and short runs of tiles of the quantizer: the
whole pipeline against the oracle, element by element."""
import numpy as np
import pytest
import torch

from paper_2306_11800_amd import synth
from test_gpu_fuzz import family, step
from test_gpu_parity import run_pipeline

pytestmark = pytest.mark.gpu

SIZES = [1, 2, 63, 255, 257, 4095, 4096, 4097, 16383, 16384, 16385, 5 * 12288 + 7]


@pytest.mark.parametrize("kind", [0, 3, 4, 5, 6, 8])
@pytest.mark.parametrize("ordered", [True, False])
def test_size_classes(monkeypatch, kind, ordered):
    from paper_2306_11800_amd import api
    monkeypatch.setenv("INSHR_NO_LDS_ORDER", "0" if ordered else "1")
    ctx = api.Context(torch.device("cuda:0"))
    rng = np.random.default_rng(700 + kind)
    sizes = SIZES if ordered else SIZES[::3] + [4096]
    prevs = [family(rng, kind, n) for n in sizes]
    curs = [step(rng, p, kind) for p in prevs]
    grid = synth.grid_paper(prune=(0.0, 0.2, 0.5), protect=(0.0, 0.005, 0.02), bins=(2, 3, 4, 6, 12, 16, 256))
    run_pipeline(ctx, prevs, curs, grid, synth.EPS_DEFAULT)
    run_pipeline(ctx, prevs[:4], curs[:4], synth.grid_small(), 1e-9, check_all_cfg_quantize=True)
    ctx.close()


def repeated(rng, kind, n):
    """Values of which one is repeated (norm weights of one, biases of zero, sparse moments)."""
    x = rng.standard_normal(n).astype(np.float32)
    if kind == "constant":
        x[:] = 1.0
    elif kind == "zero":
        x[:] = 0.0
    elif kind == "signs":
        x = np.sign(x).astype(np.float32)
    elif kind == "sparse":
        x[rng.random(n) < 0.9] = 0.0
    elif kind == "run":  # a third of the values in the midst of the positive ones
        x[rng.random(n) < 0.33] = 0.7
    else:  # "ends": the largest and the smallest
        x = np.clip(x, -0.6, 0.8).astype(np.float32)
    return x


KINDS = ["constant", "zero", "signs", "sparse", "run", "ends"]


def test_repeated_values():
    from paper_2306_11800_amd import api
    ctx = api.Context(torch.device("cuda:0"))
    rng = np.random.default_rng(701)
    sizes = [128, 129, 300, 4095, 4096, 5000, 16384]  # (a run of more than 128 in a bin is taken at once)
    prevs = [repeated(rng, kind, n) for kind in KINDS for n in sizes]
    curs = [repeated(rng, kind, n) for kind in KINDS for n in sizes]
    grid = synth.grid_paper(prune=(0.0, 0.2, 0.5), protect=(0.0, 0.005, 0.02), bins=(2, 3, 4, 6, 12, 16, 256))
    run_pipeline(ctx, prevs, curs, grid, synth.EPS_DEFAULT)
    ctx.close()


@pytest.mark.parametrize("n", [4096, 16384])
def test_time_with_repeated_values(n):
    """No lane adds a long run of equal values up by itself: the search takes at most three times what it
    takes for values that are all different (1.4 times measured; 20 to 80 times with one addition per
    value)."""
    from paper_2306_11800_amd import api
    ctx = api.Context(torch.device("cuda:0"))
    rng = np.random.default_rng(702)
    grid = synth.grid_paper(prune=(0.0, 0.1, 0.2, 0.3, 0.4))

    def ms(x):
        t = [torch.from_numpy(x).to("cuda:0")]
        ctx.search(t, grid, 0.05, want_scores=False)
        ctx.profile(True)
        for _ in range(10):
            ctx.search(t, grid, 0.05, want_scores=False)
        times = ctx.profile_read()
        ctx.profile(False)
        return sum(v[0] for v in times.values())

    base = ms(rng.standard_normal(n).astype(np.float32))
    for kind in KINDS:
        assert ms(repeated(rng, kind, n)) < 3.0 * base, kind
    ctx.close()
