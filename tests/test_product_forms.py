"""What a model's bf16 product runs on, by its sizes (bf16_form; the rule needs no GPU)."""
import ctypes

import pytest

from paper_2501_04012_amd import build

F128, F192, F256, F384, P128, P256, W288 = range(7)


@pytest.fixture(scope="module")
def form():
    f = ctypes.CDLL(build.LIB_PATH)._ZN2fc9bf16_formEiiibPKvm
    f.argtypes = [ctypes.c_int] * 3 + [ctypes.c_bool, ctypes.c_void_p, ctypes.c_size_t]
    return lambda M, N, K, packed=True, lent=0: f(M, N, K, packed, 16 if lent else None, lent)


@pytest.mark.parametrize("M,N,K", [(4753, 6912, 2304), (7185, 4608, 1536), (21777, 1536, 1536), (5393, 6144, 2048), (3601, 9216, 2304),
                                   (6801, 3072, 12288), (14481, 2304, 2304), (24349, 2880, 11520)])
@pytest.mark.parametrize("lent", [0, 64 << 20])
def test_packed_128x256_keeps_what_it_is_faster_at(form, M, N, K, lent):
    """384x192 tiles take 1.03 to 1.10 times as long here."""
    assert form(M, N, K, True, lent) == P256


@pytest.mark.parametrize("M,N,K", [(495, 8640, 2880), (6545, 576, 2304), (1169, 3456, 3456), (3601, 3456, 1152)])
def test_a_last_round_of_few_128x128_tiles(form, M, N, K):
    """A few tiles more than one, and three, to a CU that holds two: 128x288 and 384x192 tiles take 1.06 to 1.29 times as long."""
    assert form(M, N, K, False) == F128


@pytest.mark.parametrize("M,N,K", [(9489, 6912, 2304), (28945, 2304, 2304), (27921, 1728, 576)])
def test_a_last_round_of_few_256x256_tiles(form, M, N, K):
    """Two to four tiles in the last of four or five rounds: 384x192 takes 1.05 times as long."""
    assert form(M, N, K, False) == F256


@pytest.mark.parametrize("M,N,K,packed,want", [
    (8192, 1152, 4608, True, W288), (7300, 1152, 4608, True, W288), (15742, 576, 2304, True, W288), (900, 9216, 2304, True, W288),
    (8192, 1152, 1152, True, F192), (14592, 1152, 4608, True, F384), (24320, 576, 576, False, F384), (32768, 1152, 4608, True, F192),
    (9326, 6144, 2048, True, P256), (4096, 4608, 1152, True, P128), (17776, 9216, 3072, True, F256)])
def test_forms_of_products_in_use(form, M, N, K, packed, want):
    assert form(M, N, K, packed, 64 << 20) == want
