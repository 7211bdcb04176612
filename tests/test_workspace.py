"""acache_workspace_size keeps what the header promises: the size it names for
a call is enough for that call.  CPU only: calls with pointers that no launch
could use, which without a GPU end at the first launch (status 6) once every
check has passed."""

import ctypes

import pytest
import torch

# (d_model, n_heads, n_kv_heads, d_ff): the repository's two models, a wider
# layer, one with more query columns than model columns, and a small one
LAYERS = [(4096, 32, 32, 12288), (3584, 28, 4, 18944), (8192, 64, 8, 28672), (1024, 32, 8, 2048), (512, 4, 2, 768)]
WORKSPACE, DEVICE = 5, 6


@pytest.fixture(scope="module")
def A():
    if torch.cuda.is_available():
        pytest.skip("the calls would run on the GPU")
    from paper_2608_26140_amd import acache
    return acache


def _dims(A, layer):
    d, H, Hkv, F = layer
    return A.make_dims(d, H, Hkv, 128, F, "bf16")


@pytest.mark.parametrize("layer", LAYERS)
def test_decode_fits_the_size_it_names(A, layer):
    dims, p = _dims(A, layer), ctypes.c_void_p(256)
    w = A.LayerWeights(*[256] * 6)
    for batch in (1, 2, 7, 16, 24, 32, 48, 64):
        for rows in (1, 16, 33, 96, 128, 144, 160, 176, 256, 400, 512, 1024):
            if batch * rows * max(layer[0], layer[1] * 128, layer[3]) >= 1 << 31:
                continue
            for L, k in ((0, 0), (64, 8), (8192, 1638)):
                need = A.acache_workspace_size(dims, batch * rows, batch, L)
                call = lambda n: A.lib.acache_layer_decode(  # noqa: E731
                    ctypes.byref(dims), ctypes.byref(w), batch, rows, p, p, p, p, L, p, k, p, 40, p, p,
                    layer[2] * 128, 1000, p, n, None)
                assert call(need) == DEVICE, (batch, rows, L)
                assert call(need - 1) == WORKSPACE
