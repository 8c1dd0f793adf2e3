"""Products along a very long K: tiles of 128x128 as long as their rows lie within 32-bit offsets, not the plain kernel."""
import pytest

from launches import Launches
from util import record

STORE, GELU, GATE, HEADS, UNPATCH = range(5)


@pytest.mark.parametrize("K,kernel", [((1 << 22) - 64, None), (1 << 22, "k_gemm_dlds"), ((1 << 24) - 64, "k_gemm_dlds"), (1 << 24, "k_gemm_plain")])
def test_kernel_of_a_long_k(tmp_path, K, kernel):
    todo = [(mode, M, N, K, packed, lent) for mode in (STORE, GELU, GATE, HEADS, UNPATCH) for M, N in ((32, 96), (320, 384), (5000, 1152), (120000, 96), (9000, 3072))
            for packed in (False, True) for lent in (0, 1 << 30)]
    for product, (status, _, kernels) in zip(todo, Launches(tmp_path)(todo)):
        assert status == 0, product
        if kernel == "k_gemm_dlds":
            assert kernels[0] == ("k_gemm_dlds", 128, 128), (product, kernels)
        else:
            assert (kernels[0][0] == "k_gemm_plain") == (kernel is not None), (product, kernels)


@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K", [(320, 320, (1 << 22) + 64), (160, 136, (1 << 24) - 64)])
def test_linear_bf16_along_a_long_k(fc, M, N, K):
    import torch
    g = torch.Generator(device="cuda:0").manual_seed(K)
    A = torch.empty((M, K), dtype=torch.bfloat16, device="cuda:0").normal_(generator=g)
    W = torch.empty((N, K), dtype=torch.bfloat16, device="cuda:0").normal_(std=K ** -0.5, generator=g)
    want = torch.zeros((M, N), dtype=torch.float64, device="cuda:0")
    for k in range(0, K, 1 << 20):
        want += A[:, k:k + (1 << 20)].double() @ W[:, k:k + (1 << 20)].double().t().contiguous()
    out = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda:0")
    fc.fc_op_linear(fc.FC_BF16, A, W, None, None, out, M, N, K, 0)
    err = float((out.double() - want).norm() / want.norm())
    record(rel_l2=err)
    # rounding of the result to bf16: at most 2^-9 of it; K / 32 fp32 additions one after the other: 2^-24 sqrt(K / 32) in the mean
    assert err < 2.0 ** -9 + 2.0 ** -24 * (K / 32) ** 0.5
