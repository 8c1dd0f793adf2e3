"""The kernel that a bf16 product launches is the one that bf16_form names (the choice of packed weights at a model's start reads it too)."""
import random

import pytest

from launches import Launches
from test_product_forms import F128, F192, F256, F384, P128, P256, W288

GELU, GATE, HEADS = 1, 2, 3
KERNELS = {F128: ("k_gemm_dlds", 128, 128), F192: ("k_gemm_dlds", 256, 192), F256: ("k_gemm_dlds", 256, 256), F384: ("k_gemm_dlds", 384, 192),
           P256: ("k_gemm_packed", 128, 256)}


@pytest.fixture(scope="module")
def launches(tmp_path_factory):
    return Launches(tmp_path_factory.mktemp("launches"))


def products():
    """Widths in use and any others, as a model's products and alone, with what a model lends and with other amounts."""
    r = random.Random(17)
    yield GATE, 700, 1344, 5376, True, 16 << 20
    yield GELU, 1200, 3264, 13056, True, 64 << 20
    yield GATE, 2776, 5952, 23808, True, 64 << 20
    for _ in range(20000):
        M, D = round(2 ** r.uniform(8, 15.5)), 64 * (r.choice([9, 12, 16, 18, 20, 24, 32, 36, 48]) if r.random() < 0.5 else r.randrange(1, 96))
        mode, N, K = r.choice([(HEADS, 3 * D, D), (GATE, D, D), (GELU, 4 * D, D), (GATE, D, 4 * D), (GATE, 8 * r.randrange(4, 600), 64 * r.randrange(1, 80))])
        yield mode, M, N, K, r.random() < 0.7, r.choice([0, M * min(N, K) * 2, 1 << 20, 16 << 20, 64 << 20, 1 << 30])


def test_the_form_named_is_the_form_launched(launches):
    todo = [p for p in products() if -(-p[1] // 128) * -(-p[2] // 128) >= 32]        # (fewer tiles: k_gemm_skinny, before there is a choice)
    seen = set()
    for p, (status, form, kernels) in zip(todo, launches(todo)):
        assert status == 0 and kernels, p
        seen.add((form, kernels[0]))
        if form == W288:
            assert kernels[0][0] == "k_gemm_288", (p, kernels)
        elif form == P128:
            assert kernels[0] in [("k_gemm_packed", 128, 128), ("k_gemm_packed", 128, 192)], (p, kernels)
        else:
            assert kernels[0] == KERNELS[form], (p, form, kernels)
    assert len(seen) == 8, seen                            # every form, both narrow ones
