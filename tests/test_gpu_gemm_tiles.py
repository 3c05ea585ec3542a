"""GPU parity of the matrix-product kernel at every tile width its dispatch
takes (64, 96, 128 and 256 tokens, and 256-token tiles followed by narrower
ones) against the fp64 oracles, at the edges of the widths' ranges.  Bars:
those of the scorer and layer tests, where they are derived."""
import numpy as np
import pytest

from gpu_util import host_bf16_to_f64, say
from test_gpu_layer import _check_selection, _close, _oracle, _run_layer, _tiny_variant
from test_gpu_scorer import SCORE_MAX_ABS, _run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [
    # n_q, n_kv, d, La, Lb, hidden: 4 feature tiles, K loops of 3 to 16 steps
    (1, 1, 64, 0, 1, 1024),         # one token, as many K steps as LDS stages
    (2, 1, 64, 3, 65, 1024),        # 64-token tiles, one token over a tile
    (2, 1, 64, 0, 4096, 1024),      # 64: the last length of one round
    (1, 1, 64, 5, 4097, 1024),      # 96
    (1, 1, 128, 0, 6144, 1024),     # 96: the last length of one round
    (3, 1, 64, 1, 6145, 1024),      # 128, ragged
    (2, 1, 64, 0, 8192, 1024),      # 128: the last length of one round
    (4, 2, 128, 0, 8193, 1024),     # 256, one token over a tile
    (1, 1, 64, 7, 17001, 1024),     # one round of 256, then 64
])
def test_scorer_tile_widths(shape):
    say(f"[tile widths] scorer {shape}")
    got, ref, _ = _run(*shape)
    err = np.abs(got - ref)
    say(f"  max {err.max():.3e}")
    assert np.isfinite(got).all()
    assert err.max() <= SCORE_MAX_ABS


@pytest.mark.parametrize("rows", [600, 1000], ids=["96_tokens", "128_tokens"])
def test_layer_tile_widths(rows):
    # 32 feature tiles in every product: 96-token tiles fill one round at 600
    # rows, 128-token tiles at 1000 (64-token tiles: the tiny layers)
    lw = _tiny_variant(f"wide_{rows}", n_q_heads=48, n_kv_heads=8, head_dim=128, hidden=8192,
                       intermediate=4096, anchor_len=rows // 5, local_len=rows - rows // 5,
                       host_idx=1)
    say(f"[tile widths] layer of {rows} rows")
    inp, got = _run_layer(lw)
    ref = _oracle(lw, inp)
    _close(host_bf16_to_f64(got["out"]), ref["out"], "hidden_out")
    _close(host_bf16_to_f64(got["k"]), ref["k"], "K cache (post-RoPE)")
    _close(host_bf16_to_f64(got["v"]), ref["v"], "V cache")
    _check_selection(lw, inp, got, ref)
