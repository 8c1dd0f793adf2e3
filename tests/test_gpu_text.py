"""Texts of a call: aligned or not, whole pieces of four or not, with and without the guidance rows' text."""
import numpy as np
import pytest

from oracle import sampler
from paper_2501_04012_amd import synth
from util import host, record, rel_l2


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [synth.DT_F32, synth.DT_BF16])
@pytest.mark.parametrize("guidance", [False, True])
@pytest.mark.parametrize("text_len,text_dim", [(8, 64), (3, 65), (1, 4)])
def test_text_through_any_pointer(fc, dtype, guidance, text_len, text_dim):
    """A step's text from an aligned address and from one four bytes on: the oracle's noise estimate, and the same one up to the order of
    fp32 sums."""
    import torch
    cfg = synth.ModelConfig(frames=2, height=4, width=8, channels=4, patch=2, hidden=64, heads=4, mlp_dim=128, depth=1, text_len=text_len,
                            text_dim=text_dim, attn_mode=synth.ATTN_FACTORIZED_CROSS, dtype=dtype)
    W = synth.make_weights(cfg, 3, std=0.1)
    den = fc.Denoiser(cfg, W, 2, guidance)
    g = torch.Generator(device="cuda:0").manual_seed(4)
    n = text_len * text_dim
    lat = torch.randn(2, cfg.frames, cfg.height, cfg.width, cfg.channels, device="cuda:0", generator=g)
    texts = torch.randn(3 * n + 2, device="cuda:0", generator=g)

    def split(flat):
        return flat[:2 * n].reshape(2, text_len, text_dim), flat[2 * n:3 * n].reshape(text_len, text_dim) if guidance else None

    def want(flat):
        cond, null = split(host(flat))
        return sampler.denoise_step(cfg, W, host(lat), cond, null, synth.Schedule(), 25, dtype=np.float64, return_eps=True)[1]

    got = []
    for off in (0, 1):
        flat = torch.cat([texts.new_zeros(off), texts])[off:]                   # the same values, `off` floats into an allocation
        eps, x = torch.empty_like(lat), lat.clone()
        den.step(x, *split(flat), synth.Schedule(), 25, eps_out=eps)
        got.append(eps)
    torch.cuda.synchronize()
    den.close()
    expected = want(texts)
    errors = [rel_l2(host(e), expected) for e in got]
    record(aligned=errors[0], unaligned=errors[1], difference=float((got[0] - got[1]).norm() / got[0].norm()))
    # fp32 sums of up to 65 products in another order: 1e-6 of the text, less of the estimate (7.5 times a difference with guidance)
    assert float((got[0] - got[1]).norm() / got[0].norm()) < (1e-4 if dtype == synth.DT_F32 else 2e-2)
    # the estimate's error of a step in fp32, and in bf16 (3e-2 with guidance, which multiplies it)
    tolerance = 1e-4 if dtype == synth.DT_F32 else 3e-2 if guidance else 2e-2
    assert max(errors) < tolerance
    # a text read one float too early or late, and only the guidance rows' one, would show
    late = torch.cat([texts[1:], texts[:1]])
    assert rel_l2(want(late), expected) > 5 * tolerance
    if guidance:
        assert rel_l2(want(torch.cat([texts[:2 * n], late[2 * n:]])), expected) > 5 * tolerance
