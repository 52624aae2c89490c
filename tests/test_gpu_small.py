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
