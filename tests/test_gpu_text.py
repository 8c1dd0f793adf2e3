"""Texts of a call: aligned or not, whole pieces of four or not, with and without the guidance rows' text."""
import numpy as np
import pytest

from paper_2501_04012_amd import synth


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [synth.DT_F32, synth.DT_BF16])
@pytest.mark.parametrize("guidance", [False, True])
@pytest.mark.parametrize("text_len,text_dim", [(8, 64), (3, 65), (1, 4)])
def test_text_through_any_pointer(fc, dtype, guidance, text_len, text_dim):
    """A step's text from an aligned address and from one four bytes on: the same noise estimate up to the order of fp32 sums."""
    import torch
    cfg = synth.ModelConfig(frames=2, height=4, width=8, channels=4, patch=2, hidden=64, heads=4, mlp_dim=128, depth=1, text_len=text_len,
                            text_dim=text_dim, attn_mode=synth.ATTN_FACTORIZED_CROSS, dtype=dtype)
    den = fc.Denoiser(cfg, synth.make_weights(cfg, 3, std=0.1), 2, guidance)
    g = torch.Generator(device="cuda:0").manual_seed(4)
    lat = torch.randn(2, cfg.frames, cfg.height, cfg.width, cfg.channels, device="cuda:0", generator=g)
    texts = torch.randn(3 * text_len * text_dim + 2, device="cuda:0", generator=g)
    got = []
    for off in (0, 1):
        flat = torch.cat([texts.new_zeros(off), texts])[off:]                   # the same values, `off` floats into an allocation
        n = text_len * text_dim
        eps, x = torch.empty_like(lat), lat.clone()
        den.step(x, flat[:2 * n].view(2, text_len, text_dim), flat[2 * n:3 * n].view(text_len, text_dim) if guidance else None,
                 synth.Schedule(), 25, eps_out=eps)
        got.append(eps)
    torch.cuda.synchronize()
    den.close()
    assert bool(torch.isfinite(got[0]).all())
    # fp32 sums of up to 65 products in another order: 1e-6 of the text, less of the estimate (7.5 times a difference with guidance); a
    # text read at the wrong place changes it by a tenth and more
    assert float((got[0] - got[1]).norm() / got[0].norm()) < (1e-4 if dtype == synth.DT_F32 else 2e-2)
    other = texts.clone().normal_(generator=g)
    eps, x = torch.empty_like(lat), lat.clone()
    den2 = fc.Denoiser(cfg, synth.make_weights(cfg, 3, std=0.1), 2, guidance)
    den2.step(x, other[:2 * n].view(2, text_len, text_dim), other[2 * n:3 * n].view(text_len, text_dim) if guidance else None, synth.Schedule(), 25,
              eps_out=eps)
    torch.cuda.synchronize()
    den2.close()
    assert float((eps - got[0]).norm() / got[0].norm()) > 1e-3
