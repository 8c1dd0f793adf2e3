"""Steps of small fp32 models without guidance, whose last launch updates the latents itself: with and without the noise estimate handed
out, both samplers, rows that end inside a workgroup, text rows in the sequence."""
import numpy as np
import pytest
import torch

from oracle import sampler
from paper_2501_04012_amd import synth
from util import cached_weights, record, rel_l2


@pytest.mark.gpu
@pytest.mark.parametrize("mode,frames,height,width,channels,depth,requests,euler", [
    (synth.ATTN_FACTORIZED_CROSS, 4, 8, 8, 4, 1, 1, False), (synth.ATTN_FACTORIZED_CROSS, 3, 10, 6, 3, 2, 3, True),
    (synth.ATTN_FULL3D_CONCAT, 3, 6, 10, 4, 1, 2, False), (synth.ATTN_FULL3D_CONCAT, 1, 4, 6, 5, 2, 1, True)])
def test_update_in_the_last_launch(fc, mode, frames, height, width, channels, depth, requests, euler):
    cfg = synth.ModelConfig(frames=frames, height=height, width=width, channels=channels, patch=2, hidden=64, heads=4, mlp_dim=256,
                            depth=depth, text_len=7, text_dim=32, attn_mode=mode, dtype=synth.DT_F32)
    W = cached_weights(cfg, 3)
    lat = np.stack([synth.make_latent(cfg, 20 + r) for r in range(requests)]).reshape(requests, frames, height, width, channels)
    cond = np.stack([synth.make_text(cfg, 40 + r) for r in range(requests)]).reshape(requests, cfg.text_len, cfg.text_dim)
    sched = synth.Schedule(sampler=synth.SAMPLER_FLOW_EULER if euler else synth.SAMPLER_DDIM)
    den = fc.Denoiser(cfg, W, requests, False)
    texts, got = torch.from_numpy(cond).cuda(), []
    eps = torch.full(lat.shape, float("nan"), device="cuda")
    for out in (None, eps):
        x = torch.from_numpy(lat).cuda()
        den.step(x, texts, None, sched, 25, **({} if out is None else {"eps_out": out}))
        got.append(x.cpu().numpy())
    den.close()
    want, weps = sampler.denoise_step(cfg, W, lat, cond, None, sched, 25, dtype=np.float64, return_eps=True)
    record(latent_rel_l2=rel_l2(got[0], want), eps_rel_l2=rel_l2(eps.cpu().numpy(), weps))
    assert np.array_equal(got[0], got[1])
    assert rel_l2(got[0], want) <= 1e-4 and rel_l2(eps.cpu().numpy(), weps) <= 1e-4       # the bar of an fp32 step
