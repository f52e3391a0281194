"""Size of the workspace: the records of partials lie in the area of the split + merge kernels' partials and are no more
than the blocks of a launch need."""
import ctypes as C

import pytest

# (layers, sequences, query heads, KV heads, budget, window, prompt) of 128 x bf16 rows, and the bytes of a library
# whose records had an area of their own, three per unit
SIZES = [((28, 32, 28, 4, 2048, 64, 2048), 187231488), ((28, 1024, 28, 4, 2048, 64, 2048), 5989363968),
         ((1, 1, 8, 8, 96, 16, 60), 2551552), ((2, 48, 28, 4, 500, 32, 400), 80672000),
         ((1, 4, 40, 8, 16448, 64, 16384), 113747968), ((4, 64, 32, 8, 256, 32, 256), 181177344)]


@pytest.mark.parametrize("shape,most", SIZES)
def test_workspace_size(lazyev_lib, shape, most):
    L, S, Hq, H, B, W, P = shape
    cfg = lazyev_lib.Config(n_layers=L, batch=S, n_q_heads=Hq, n_kv_heads=H, head_dim=128, budget=B, window=W, prompt_len=P,
                            alpha=0.01, softmax_scale=0.0, dtype=lazyev_lib.DTYPE_BF16, score_flags=3)
    assert 0 < lazyev_lib.lib.lazyev_workspace_size(C.byref(cfg)) <= most
