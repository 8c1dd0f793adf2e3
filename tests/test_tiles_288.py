"""Products in tiles of 128 x 288 (k_gemm_288): what the compiler made of the waits, and the results at the edges."""
import math

import numpy as np
import pytest

from test_lds_dma_waits import early_barriers, listings       # noqa: F401  (a fixture)


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
