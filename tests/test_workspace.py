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


@pytest.mark.parametrize("layer", LAYERS)
def test_a_workspace_serves_fewer_rows(A, layer):
    """Every row count up to 6000 and a spread up to 40,000: more rows never
    need less."""
    dims = _dims(A, layer)
    rows = list(range(1, 6000)) + list(range(6000, 40000, 37))
    sizes = [A.acache_workspace_size(dims, r, 4, 1024) for r in rows]
    shrinks = [(a, b) for a, b, x, y in zip(rows, rows[1:], sizes, sizes[1:]) if y < x]
    assert not shrinks, shrinks[:3]


@pytest.mark.parametrize("layer", LAYERS)
def test_refresh_and_score_fit_the_size_they_name(A, layer):
    """acache_layer_recompute and acache_layer_score (the masked rows' queries
    alone) at row counts on both sides of every 64, with the size named for
    them and with that of twice the rows."""
    dims, p = _dims(A, layer), ctypes.c_void_p(256)
    w = A.LayerWeights(*[256] * 6)
    for tiles in (1, 2, 3, 4, 5, 9, 24, 36, 72, 80, 85, 106, 128, 145, 200):
        for rows in (64 * tiles - 1, 64 * tiles, 64 * tiles + 1):
            cu = (ctypes.c_int32 * 2)(0, rows)
            rg = A.Ragged(1, cu, (ctypes.c_int32 * 2)(0, rows + 100))
            sa = A.ScoreArgs(256, cu, 256, 100, A.ACACHE_NORM_AFFIX, 256)
            for size in (A.acache_workspace_size(dims, rows, 1, 100), A.acache_workspace_size(dims, 2 * rows, 1, 100)):
                args = (ctypes.byref(dims), ctypes.byref(w), ctypes.byref(rg), p, p, p, p, p, p, layer[2] * 128, 1000)
                assert A.lib.acache_layer_recompute(*args, None, p, size, None) == DEVICE, rows
                if layer[3] >= layer[0]:
                    assert A.lib.acache_layer_score(*args, ctypes.byref(sa), p, size, None) == DEVICE, rows
