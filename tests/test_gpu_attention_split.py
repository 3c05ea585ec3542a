"""GPU parity of the two forms of the attention kernel against the fp64 oracle,
every row, at the attention test's bar.  The key-split form (at most 256
workgroups of 256 rows, keys past one tile): edges of its 128-row workgroups and
its tiles, a second group with one key or none, tiles over two and over many
segments.  The 256-row form on ragged shapes, with enough query heads that it
is the one taken.  Both with the running max moving late (softmax scale 1.0)."""
import pytest

import oracle
from paper_2502_12085_amd import inputs
from gpu_util import (O_REL_PEAKED, assert_attention_close, host_bf16_to_f64, need_gpu,
                      run_attention, say, upload)

pytestmark = pytest.mark.gpu

SPLIT = [
    # n_hosts, host_idx, La, Lb, l_p, n_q, n_kv, d
    (1, 0, 0, 65, 0, 2, 1, 128),        # the second group's tile holds one key
    (1, 0, 0, 64, 0, 2, 1, 128),        # one tile: the 256-row form
    (1, 0, 0, 129, 0, 2, 1, 64),
    (1, 0, 0, 128, 0, 2, 1, 64),        # one tile: the 256-row form
    (4, 3, 1, 67, 67, 1, 1, 128),       # one anchor row, every row passed on
    (1, 0, 0, 193, 0, 4, 2, 128),       # four tiles for the last rows, one for the first
    (3, 2, 60, 67, 40, 3, 1, 128),      # 127 rows
    (3, 2, 60, 68, 64, 3, 1, 64),       # 128 rows
    (3, 2, 60, 69, 64, 3, 3, 128),      # 129 rows
    (8, 7, 33, 300, 5, 4, 2, 128),      # tiles over many passing slots
    (8, 7, 33, 300, 3, 4, 1, 64),
    (4, 3, 301, 1023, 127, 8, 2, 128),  # ragged everywhere, 27 tiles
    (4, 3, 301, 1023, 127, 8, 2, 64),
    (2, 1, 0, 700, 700, 16, 8, 128),    # no anchor, XCD-mapped heads
]
# 88 heads x 3 tiles of 256 rows = 264 workgroups; 257 heads x 1
WIDE = [
    (4, 3, 77, 524, 37, 88, 11, 128),
    (4, 3, 77, 524, 37, 88, 11, 64),
    (8, 7, 0, 513, 9, 88, 8, 128),
    (2, 1, 20, 81, 30, 257, 257, 128),
    (2, 1, 20, 81, 30, 257, 257, 64),
]


def _check(shape, scale=0.0):
    need_gpu()
    p = inputs.Problem(*shape)
    say(f"[attention forms] {p} scale {scale}")
    inp = inputs.make_inputs(inputs.Workload("forms", p), seed=41)
    o, lse = run_attention(p, upload(inp), scale)
    kw = dict(scale=scale) if scale else {}
    o_ref, lse_ref = oracle.attention_ref(inp["q"], inp["k"], inp["v"], inp["k_pass"],
                                          inp["v_pass"], anchor_len=p.anchor_len, **kw)
    assert_attention_close(host_bf16_to_f64(o), lse.cpu().numpy(), o_ref, lse_ref, str(shape),
                           **(dict(o_rel=O_REL_PEAKED) if scale else {}))


@pytest.mark.parametrize("shape", SPLIT, ids=str)
def test_key_split_form(shape):
    _check(shape)


@pytest.mark.parametrize("shape", WIDE, ids=str)
def test_row_form(shape):
    _check(shape)


@pytest.mark.parametrize("shape", [SPLIT[9], SPLIT[11], SPLIT[12], WIDE[0], WIDE[1]], ids=str)
def test_late_max(shape):
    _check(shape, 1.0)


@pytest.mark.parametrize("shape", [
    (2, 1, 0, 700, 1, 4, 1, 64),
    (4, 3, 50, 600, 40, 4, 1, 64),
    (4, 3, 50, 600, 40, 2, 1, 128),
    (1, 0, 0, 700, 0, 2, 1, 128),
], ids=str)
@pytest.mark.parametrize("row", [390, 460, -1])
def test_values_past_the_last_tile_are_not_used(shape, row):
    # An infinite value makes NaN of the masked products of its 128-key tile,
    # and of no rows whose 256-row block ends before that tile.
    torch = need_gpu()
    p = inputs.Problem(*shape)
    say(f"[attention forms] {p} infinite value in row {row}")
    dv = upload(inputs.make_inputs(inputs.Workload("forms", p), seed=41))
    clean = run_attention(p, dv)
    row %= p.rows
    dv["v"][:, row] = float("inf")
    o, lse = run_attention(p, dv)
    end = lambda r: (r if r < p.anchor_len else r + p.passing_rows) + 1  # noqa: E731
    key = end(row) - 1
    before = [r for r in range(p.rows)
              if -(-end(min(r // 256 * 256 + 255, p.rows - 1)) // 128) * 128 <= key]
    assert before
    assert torch.equal(o[:, before], clean[0][:, before])
    assert torch.equal(lse, clean[1])
    assert torch.isinf(o[:, row]).all() or torch.isnan(o[:, row]).all()
