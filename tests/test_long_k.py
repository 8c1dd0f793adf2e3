"""Products along a very long K, in tiles of 128x128 as long as their rows lie within 32-bit offsets and not in the plain kernel, and of
operands of more than 4 GB in every other tile of the product kernel."""
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
    # rounding of normal values to bf16: 1.66e-3 of them in the root mean square; K / 32 fp32 additions one after the other: 2^-24 sqrt(K / 32) in the mean
    assert err < 2.0 ** -9 + 2.0 ** -24 * (K / 32) ** 0.5


BEYOND = [(65600 + 37, 1152, 32768, (256, 192)), (65600 + 37, 2048, 32768, (256, 256)), (2048 + 1, 65640, 32768, (256, 256))]       # M, N, K, tile


@pytest.mark.parametrize("M,N,K,tile", BEYOND)
def test_tiles_of_the_large_operands(tmp_path, M, N, K, tile):
    assert max(M, N) * K * 2 >= 2 ** 32
    (status, _, launched), = Launches(tmp_path)([(STORE, M, N, K, False, 0)])
    assert status == 0 and launched == [("k_gemm_dlds", *tile)]


@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K", [b[:3] for b in BEYOND])
def test_linear_bf16_of_large_operands_in_three_stages(fc, M, N, K):
    """Rows and columns at the ends and around 2^31 and 2^32 bytes against the float64 product, the rest for finiteness."""
    import torch
    g = torch.Generator(device="cuda:0").manual_seed(M)
    A = torch.empty((M, K), dtype=torch.bfloat16, device="cuda:0").normal_(generator=g)
    W = torch.empty((N, K), dtype=torch.bfloat16, device="cuda:0").normal_(std=K ** -0.5, generator=g)
    out = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda:0")
    fc.fc_op_linear(fc.FC_BF16, A, W, None, None, out, M, N, K, 0)
    assert bool(torch.isfinite(out).all())
    pick = lambda n: torch.tensor(sorted({x for e in (0, 256, 32768, 65536, n) for x in range(e - 3, e + 3) if 0 <= x < n} | set(range(0, n, 997))), device="cuda:0")
    m, n = pick(M), pick(N)
    want = A[m].double() @ W.double().t().contiguous() if N < M else (W[n].double() @ A.double().t().contiguous()).t()
    got = out[m].double() if N < M else out[:, n].double()
    err = float((got - want).norm() / want.norm())
    record(rel_l2=err)
    # rounding as above; element by element half an ulp of the bf16 result, and fp32 sums of 1024 instructions one after the other
    assert err < 2.0 ** -9 and bool(((got - want).abs() <= 2.0 ** -8 * want.abs() + 1e-4).all())
