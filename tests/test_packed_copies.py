"""The products of a model's blocks run in packed tiles wherever bf16_form names them for the scratch memory that the model lends: it holds
the packed copies that this takes."""
import subprocess

import pytest

from launches import STUBS, kernels, program
from test_launched_form import KERNELS
from test_product_forms import P128, W288, form            # noqa: F401  (a fixture)

SOURCE = STUBS + r"""
#include <cstdlib>
#include "flexdenoise.h"
int main() {
  fc_model_config c{};
  c.channels = 4; c.patch = 2; c.depth = 1; c.text_len = 8; c.text_dim = 64; c.t_embed_dim = 64; c.attn_mode = FC_ATTN_FACTORIZED_CROSS; c.dtype = FC_BF16; c.ln_eps = 1e-6f;
  int requests;
  while (scanf("%d %d %d %d %d %d %d", &c.frames, &c.height, &c.width, &c.hidden, &c.heads, &c.mlp_dim, &requests) == 7) {
    fc_model* m = nullptr;
    size_t n = 0, bytes = 0;
    fc_schedule s{1000, 1e-4f, 0.02f, 50, 1.0f, 0.0f, FC_SAMPLER_DDIM, 0};
    int rc = fc_model_create(&c, &m);
    if (rc == FC_OK) rc = fc_model_weight_count(m, &n);
    float* blob = (float*)calloc(n, 4);                  // never read
    if (rc == FC_OK) rc = fc_model_set_weights(m, blob, n);
    if (rc == FC_OK) rc = fc_workspace_bytes(m, requests, 0, &bytes);
    seen.clear();
    if (rc == FC_OK) rc = fc_denoise_step(m, (float*)4096, (float*)4096, nullptr, &s, 10, requests, nullptr, (void*)4096, bytes, nullptr);
    printf("%d%s\n", rc, seen.c_str());
    fc_model_destroy(m);
    free(blob);
  }
}
"""
MODELS = [  # frames, height, width, hidden, heads, mlp_dim, requests
    (23, 60, 64, 384, 6, 3392, 1),                         # fc2 in packed tiles, but in 384x192 with more scratch memory than the model lends
    (16, 32, 32, 1152, 16, 4608, 1), (16, 32, 32, 1152, 16, 4608, 2), (15, 34, 32, 1152, 16, 1152, 1), (8, 40, 50, 576, 8, 576, 1),
    (9, 48, 48, 768, 12, 3072, 3), (13, 48, 62, 1536, 24, 6144, 1), (16, 64, 64, 1024, 16, 4096, 2)]


@pytest.fixture(scope="module")
def steps(tmp_path_factory):
    text = "".join(" ".join(map(str, m)) + "\n" for m in MODELS)
    exe = program(tmp_path_factory.mktemp("steps"), SOURCE)
    out = subprocess.run([exe], input=text, check=True, capture_output=True, text=True).stdout.splitlines()
    assert len(out) == len(MODELS)
    return {m: (int(line.split()[0]), kernels(line.split()[1:])) for m, line in zip(MODELS, out)}


@pytest.mark.parametrize("model", MODELS, ids="-".join(["%s"] * 7).__mod__)
def test_products_of_a_step(steps, form, model):           # noqa: F811
    frames, height, width, hidden, _, mlp, requests = model
    status, launched = steps[model]
    assert status == 0
    rows = requests * frames * (height // 2) * (width // 2)
    act, hid = rows * hidden * 2, rows * mlp * 2
    block = [(3 * hidden, hidden, hid), (hidden, hidden, act)] * 2 + [(hidden, hidden, 0), (hidden, hidden, act), (mlp, hidden, act), (hidden, mlp, act)]
    tiles = [k for k in launched if k[0] in ("k_gemm_dlds", "k_gemm_packed", "k_gemm_288")][:len(block)]       # (the text's products are skinny ones)
    want = [form(rows, n, k, True, lent) for n, k, lent in block]
    for product, f, kernel in zip(block, want, tiles):
        if f == W288:
            assert kernel[0] == "k_gemm_288", product
        elif f == P128:
            assert kernel[0] == "k_gemm_packed" and kernel[2] in (128, 192), (product, kernel)
        else:
            assert kernel == KERNELS[f], (product, kernel)
    assert len(tiles) == len(block)
