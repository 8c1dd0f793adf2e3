"""Narrow packed tiles (128x128 and 128x192) in a model's products, with rows and columns that end inside a tile, against the oracle."""
import numpy as np
import pytest
import torch                                              # noqa: F401  (first: the library runs on the HIP runtime that torch brings)

from launches import Launches
from oracle import sampler
from paper_2501_04012_amd import synth
from test_product_forms import P128, form                     # noqa: F401  (a fixture)
from util import cached_weights, record, rel_l2, run_step_gpu

GATE = 2
CASES = [  # hidden, heads, frames, height, width, mlp, columns of the out-projections' tiles
    (1152, 16, 16, 32, 32, 1152, 192),                        # 4096 x 1152 x 1152
    (1152, 16, 15, 34, 32, 1152, 192),                        # 4080 rows: the last tile of rows is not whole
    (1088, 17, 8, 40, 50, 1088, 192),                         # 4000 x 1088 x 1088: 17 K tiles, the last tile of columns two thirds
    (832, 13, 9, 48, 48, 832, 192),                           # 5184 x 832 x 832: 13 K tiles, the last tile of columns one third
    (576, 8, 8, 40, 50, 576, 128)]                            # 4000 x 576 x 576: an odd number of K tiles, 4.5 tiles of columns


@pytest.mark.parametrize("hidden,heads,frames,height,width,mlp,columns", CASES)
def test_the_tile_that_runs(tmp_path, form, hidden, heads, frames, height, width, mlp, columns):    # noqa: F811
    rows = frames * (height // 2) * (width // 2)
    assert form(rows, hidden, hidden, True, rows * hidden * 2) == P128
    (status, _, launched), = Launches(tmp_path)([(GATE, rows, hidden, hidden, True, rows * hidden * 2)])
    assert status == 0 and launched == [("k_gemm_packed", 128, columns)]


@pytest.mark.gpu
@pytest.mark.parametrize("hidden,heads,frames,height,width,mlp", [c[:6] for c in CASES])
def test_narrow_packed_tiles(fc, form, hidden, heads, frames, height, width, mlp):    # noqa: F811
    rows = frames * (height // 2) * (width // 2)
    assert form(rows, hidden, hidden, True, rows * hidden * 2) == P128
    cfg = synth.ModelConfig(frames=frames, height=height, width=width, channels=4, patch=2, hidden=hidden, heads=heads, mlp_dim=mlp, depth=1,
                            text_len=9, text_dim=64, attn_mode=synth.ATTN_FACTORIZED_CROSS, dtype=synth.DT_BF16)
    w = synth.Workload("narrow", cfg, weight_seed=5, latent_seed=6, text_seed=7, null_seed=None, requests=1)
    W = cached_weights(cfg, 5)
    lat, cond, null = synth.workload_inputs(w)
    got, eps = run_step_gpu(fc, w, weights=W, inputs=(lat, cond, null))
    want, weps = sampler.denoise_step(cfg, W, lat, cond, null, w.schedule, w.step, dtype=np.float64, return_eps=True)
    record(latent_rel_l2=rel_l2(got, want), eps_rel_l2=rel_l2(eps, weps))
    assert rel_l2(got, want) <= 1e-2 and rel_l2(eps, weps) <= 2e-2          # the bar of a bf16 step
