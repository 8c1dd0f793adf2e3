"""Products in tiles of 128 x 288 (k_gemm_288) and of 384 x 192: what the compiler made of the waits, and the results at the edges."""
import math

import numpy as np
import pytest

from oracle import sampler
from paper_2501_04012_amd import synth
from test_lds_dma_waits import early_barriers, listings       # noqa: F401  (a fixture)
from test_product_forms import F384, W288, form               # noqa: F401  (a fixture)
from util import cached_weights, record, rel_l2, run_step_gpu


def test_stages_have_landed_before_they_are_read(listings):    # noqa: F811
    """A stage, requested two ahead, has landed at the second barrier after its request."""
    names = [n for n in listings if "k_gemm_288" in n]
    assert len(names) == 3
    for name in names:
        assert sum(op == "s_barrier" for op, _, _ in listings[name]) >= 5, name
        assert not early_barriers(listings[name], True), name


@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K", [
    (7681, 1152, 4608), (8192, 1152, 4608),                   # one row in the last tile; whole tiles
    (7700, 1152, 4672), (900, 9216, 2112), (15742, 576, 2304),              # an odd number of K tiles; 33 of them; ragged rows
    (14592, 1152, 4608)])                                     # 384x192 tiles, a product of fewer than 600 of 256x256
@pytest.mark.parametrize("epilogue", [1, 2])
def test_linear_in_tiles_that_fill_the_chip(fc, M, N, K, epilogue):
    import torch
    g = torch.Generator(device="cuda:0").manual_seed(M + N + K)
    A = torch.randn(M, K, device="cuda:0", generator=g).bfloat16()
    W = (torch.randn(N, K, device="cuda:0", generator=g) / math.sqrt(K)).bfloat16()
    b, gate = torch.randn(N, device="cuda:0", generator=g), torch.randn(N, device="cuda:0", generator=g)
    want = A.double() @ W.double().t() + b.double()
    want = 0.5 * want * (1 + torch.tanh(math.sqrt(2 / math.pi) * (want + 0.044715 * want ** 3))) if epilogue == 1 else want * gate.double()
    out = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda:0")
    args = (fc.FC_BF16, A, W, b, gate if epilogue == 2 else None, out, M, N, K, epilogue)
    fc.fc_op_linear(*args)
    torch.cuda.synchronize()
    # bf16 rounds the result by up to 2^-9 of it (1.7e-3 in the mean); the fp32 sums before it are good to 1e-6
    err = (out.double() - want).norm(dim=1) / want.norm(dim=1)
    assert float(err.max()) < 4e-3, (float(err.max()), int(err.argmax()))
    assert np.isfinite(float(err.sum()))


@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K,fewer", [
    (8192, 1152, 4608, 2000), (7681, 1152, 4608, 1000), (15742, 576, 2304, 6001), (900, 9216, 2112, 257), (2900, 2880, 2880, 1300),
    (14592, 1152, 4608, 4096)])                               # 384x192 tiles, and of 128x288
@pytest.mark.parametrize("epilogue", [1, 2])
def test_rows_do_not_depend_on_their_number(fc, M, N, K, fewer, epilogue):
    """Without scratch no product of more than a few tiles adds its sums in parts: its first rows alone, in other tiles, get the same bits."""
    import torch
    g = torch.Generator(device="cuda:0").manual_seed(M + N + K)
    A = torch.randn(M, K, device="cuda:0", generator=g).bfloat16()
    W = (torch.randn(N, K, device="cuda:0", generator=g) / math.sqrt(K)).bfloat16()
    b, gate = torch.randn(N, device="cuda:0", generator=g), torch.randn(N, device="cuda:0", generator=g)
    got = []
    for rows in (M, fewer):
        out = torch.full((rows, N), float("nan"), dtype=torch.bfloat16, device="cuda:0")
        fc.fc_op_linear(fc.FC_BF16, A, W, b, gate if epilogue == 2 else None, out, rows, N, K, epilogue)
        got.append(out)
    torch.cuda.synchronize()
    assert bool(torch.isfinite(got[0].float()).all())
    assert torch.equal(got[0][:fewer], got[1])


@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K", [(9401, 1728, 576), (24321, 576, 576), (5101, 3456, 1152), (3700, 4608, 1152), (13400, 1152, 4608)])
@pytest.mark.parametrize("epilogue", [1, 2])
def test_linear_in_384x192_tiles_with_ragged_rows(fc, form, M, N, K, epilogue):    # noqa: F811
    """And an odd number of K tiles (576)."""
    assert form(M, N, K, False) == F384
    test_linear_in_tiles_that_fill_the_chip(fc, M, N, K, epilogue)


@pytest.mark.gpu
@pytest.mark.parametrize("hidden,heads,frames,height,width,requests,want", [
    (2304, 32, 5, 18, 26, 2, W288),                           # 1170 rows of two requests: 9.1 tiles of 128
    (576, 8, 19, 44, 46, 1, F384),                            # 9614 rows: 25.04 tiles of 384
    (1152, 16, 9, 48, 48, 1, F384)])                          # 5184 rows: 13.5
def test_heads_out_of_tiles_that_fill_the_chip(fc, form, hidden, heads, frames, height, width, requests, want):    # noqa: F811
    """Queries, keys and values of a step whose rows end inside a tile, against the oracle; every patch's noise estimate on its own, as a
    tile gone wrong would show in its rows."""
    cfg = synth.ModelConfig(frames=frames, height=height, width=width, channels=4, patch=2, hidden=hidden, heads=heads, mlp_dim=hidden,
                            depth=1, text_len=9, text_dim=64, attn_mode=synth.ATTN_FACTORIZED_CROSS, dtype=synth.DT_BF16)
    rows = requests * frames * (height // 2) * (width // 2)
    for lent in (0, 64 << 20):
        assert form(rows, 3 * hidden, hidden, hidden % 128 == 0, lent) == want
    w = synth.Workload("heads", cfg, weight_seed=5, latent_seed=6, text_seed=7, null_seed=None, requests=requests)
    W = cached_weights(cfg, 5)
    lat, cond, null = synth.workload_inputs(w)
    got, eps = run_step_gpu(fc, w, weights=W, inputs=(lat, cond, null))
    want_lat, weps = sampler.denoise_step(cfg, W, lat, cond, null, w.schedule, w.step, dtype=np.float64, return_eps=True)
    patches = lambda x: np.asarray(x, np.float64).reshape(requests, frames, height // 2, 2, width // 2, 2, 4).transpose(0, 1, 2, 4, 3, 5, 6).reshape(-1, 16)
    d = np.linalg.norm(patches(eps) - patches(weps), axis=1) / np.linalg.norm(patches(weps), axis=1)
    record(latent_rel_l2=rel_l2(got, want_lat), eps_rel_l2=rel_l2(eps, weps), worst_patch=float(d.max()))
    # bf16 against float64: 1e-2 of the latent and 2e-2 of the estimate are the bar of a step; a patch has 4 % (test_bf16_model_with_packed_weights)
    assert rel_l2(got, want_lat) <= 1e-2 and rel_l2(eps, weps) <= 2e-2
    assert d.max() < 4e-2
