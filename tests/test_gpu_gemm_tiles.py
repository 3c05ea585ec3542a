"""GPU parity of the matrix-product kernel at every tile width its dispatch
takes (64, 96, 128 and 256 tokens, and 256-token tiles followed by narrower
ones) against the fp64 oracles, at the edges of the widths' ranges.  Bars:
those of the scorer and layer tests, where they are derived."""
import numpy as np
import pytest

from paper_2502_12085_amd import inputs
from gpu_util import dev_bf16, host_bf16_to_f64, need_gpu, say
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
    (1, 1, 64, 7, 17001, 1024),     # three rounds of 96
    (1, 1, 64, 7, 18500, 1024),     # one round of 256, then 64, the last of 4 tokens
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


@pytest.mark.parametrize("d, lb, hidden", [
    (64, 200, 1024),     # 64-token tiles, the last of 8 tokens
    (128, 5000, 1024),   # 96
    (64, 8192, 1024),    # 128
    (64, 17001, 1024),   # 96 in three rounds
    (64, 18500, 1024),   # 256, then 64
    (64, 20500, 1024),   # 256, then 96
    (128, 9000, 256),    # 64 in one feature tile
])
def test_equal_tokens_score_alike(d, lb, hidden):
    # every local row holds the same token: the compressor's tie rule takes the
    # lower index of equal scores, so a token's sums may not depend on its tile
    say(f"[tile widths] one token {lb} times, hidden {hidden}")
    one, _, _ = _run(1, 1, d, 0, 1, hidden)
    torch = need_gpu()
    from paper_2502_12085_amd import apb
    rng = np.random.default_rng(0)
    q, k, v = (dev_bf16(inputs.f32_to_bf16_bits(rng.standard_normal((1, 1, d)).astype(np.float32)))
               .expand(1, lb, d).contiguous() for _ in range(3))
    w = inputs.make_scorer_weights(1, 1, d, hidden, 0)
    f = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    p = apb.ScorerProblem(0, lb, 1, 1, d, hidden)
    ws = torch.empty(apb.scorer_workspace_size(p), dtype=torch.uint8, device="cuda")
    s = torch.full((1, lb), float("nan"), dtype=torch.float32, device="cuda")
    apb.retaining_scores(p, q, k, v, dev_bf16(w["w1"]), f(w["b1"]), f(w["w2"]), f(w["b2"]), s, ws)
    got = s.cpu().numpy().astype(np.float64)
    say(f"  distinct scores {np.unique(got).size}, spread {got.max() - got.min():.1e}")
    assert (got == one[0, 0]).all()  # and the score it has alone
