"""GPU parity of the decoding step for 65 to 127 rows per KV head, where two
groups of four waves share a workgroup and meet in LDS, against the fp64
oracle at the decode test's bar: every count of row blocks and of waves
without rows, splits whose groups own unequal numbers of key blocks (one, and
none for the second group, in the last split), masked new tokens, both head
sizes, and the running max moving late (softmax scale 1.0) by other amounts in
the two groups."""
import numpy as np
import pytest

import oracle
from paper_2502_12085_amd import inputs
from gpu_util import O_REL_PEAKED, assert_attention_close, need_gpu, say
from test_gpu_decode import _run_decode

pytestmark = pytest.mark.gpu


# n_q, n_kv, d, Lc, n_new, append; softmax scale
ONE_LAUNCH = [
    ((8, 2, 128, 127, 1, 1), 0.0),       # four blocks, one per group
    ((8, 2, 128, 150, 3, 0), 0.0),       # five: the second turn is one group's
    ((32, 8, 128, 383, 1, 1), 0.0),      # 12 blocks
    ((32, 8, 128, 384, 1, 1), 0.0),      # 13: split and merge
    ((4, 1, 64, 97, 2, 1), 0.0),         # four blocks, four groups without any
    ((4, 1, 64, 894, 2, 1), 0.0),        # 28 blocks
    ((4, 1, 64, 895, 2, 1), 0.0),        # 29: split and merge
    ((4, 1, 64, 1022, 2, 1), 0.0),       # 32
    ((4, 1, 64, 1023, 2, 1), 0.0),       # 33
    ((10, 2, 64, 700, 10, 1), 0.0),      # 50 rows: two row blocks
    ((24, 2, 128, 200, 10, 0), 0.0),     # 120 rows in four row blocks
    ((8, 2, 128, 40, 1, 1), 0.0),        # two blocks: one split of one group
    ((8, 2, 128, 350, 2, 1), 1.0),
    ((4, 1, 64, 900, 3, 1), 1.0),
]


GROUPS = [
    ((32, 16, 64, 3200, 33, 1), 0.0),    # 66 rows: the third row block has two
    ((48, 16, 128, 5000, 25, 0), 0.0),   # 75 rows, 157 blocks in splits of 10
    ((64, 16, 128, 4400, 31, 1), 0.0),   # 124 rows: four row blocks
    ((40, 8, 128, 9300, 17, 1), 0.0),    # 85 rows, GQA 5, last split of two blocks
    ((14, 2, 64, 15380, 18, 0), 0.0),    # 126 rows, two heads, last split of one block
    ((127, 127, 64, 200, 100, 1), 0.0),  # one split per head, new tokens longer than a block
    ((32, 16, 128, 5000, 33, 1), 1.0),
    ((8, 2, 64, 15990, 31, 1), 1.0),
]
# As many rows over shorter splits: a workgroup per row block.
SHORT = [
    ((32, 16, 64, 2100, 33, 1), 0.0),
    ((48, 16, 128, 2500, 25, 0), 0.0),
    ((64, 16, 128, 2049, 31, 1), 0.0),
    ((40, 8, 128, 4500, 17, 1), 0.0),
    ((32, 16, 128, 2100, 33, 1), 1.0),
]


@pytest.mark.parametrize("shape, scale", ONE_LAUNCH + GROUPS + SHORT)
def test_decode_wave_groups(shape, scale):
    need_gpu()
    n_q, n_kv, d, lc, n_new, app = shape
    say(f"[decode groups] {shape} scale {scale}")
    case = inputs.make_decode_case(n_q, n_kv, d, [lc], n_new, seed=23)
    kc, vc = case["caches"][0]
    kn = case["k_new"] if app else None
    vn = case["v_new"] if app else None
    o, lse = _run_decode(case["q"], kc, vc, kn, vn, n_q, n_kv, d, scale)
    kw = dict(scale=scale) if scale else {}
    o_ref, lse_ref = oracle.decode_attention_ref(case["q"], kc, vc, kn, vn, **kw)
    assert_attention_close(o, lse, o_ref, lse_ref, f"decode groups {shape}",
                           **(dict(o_rel=O_REL_PEAKED) if scale else {}))


@pytest.mark.parametrize("d", [64, 128])
def test_decode_without_keys(d):
    q = inputs.make_decode_case(4, 2, d, [1], 3, seed=1)["q"]
    empty = np.zeros((2, 0, d), np.uint16)
    o, lse = _run_decode(q, empty, empty, None, None, 4, 2, d)
    assert (o == 0).all() and np.isneginf(lse).all()


@pytest.mark.parametrize("d, cache, n_new, first, last, o_nan", [
    (128, 20, 2, 3, 3, False),           # one split, which has the NaN
    (64, 40, 2, 33, 33, False),
    (128, 100, 1, 3, 3, True),           # one launch, a group of four
    (64, 250, 3, 100, 100, True),
    (128, 100, 1, 0, 99, False),         # all of them
    (64, 250, 3, 0, 249, False),
    (128, 36000, 25, 100, 100, True),    # 100 rows: two groups, one with the NaN
])
def test_decode_with_nan_keys(d, cache, n_new, first, last, o_nan):
    # A part of the keys whose logits are NaN has no LSE.  It is no part of the
    # row's LSE, and the row's output is NaN unless no other part is left: then
    # it is that of a host without keys.
    n_q, n_kv = 8, 2
    say(f"[decode groups] NaN in keys {first} to {last} of {cache}, d {d}")
    case = inputs.make_decode_case(n_q, n_kv, d, [cache], n_new, seed=5)
    kc, vc = case["caches"][0]
    kc[:, first:last + 1] = 0x7fc0
    o, lse = _run_decode(case["q"], kc, vc, None, None, n_q, n_kv, d)
    if o_nan:
        assert np.isnan(o).all() and np.isfinite(lse).all()
    else:
        assert (o == 0).all() and np.isneginf(lse).all()
