"""Which form of a kernel the host chooses (``csrc/apb_plan.h``, plain C++): the
forms that the GPU tests' shapes are written for are the ones they run, and the
rules hold where a form that was measured slower would be taken."""
import os
import subprocess

import pytest

import test_gpu_attention_split as attention_forms
import test_gpu_decode_groups as decode_forms
import test_zz_no_alloc as no_alloc
from paper_2502_12085_amd import apb

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2502_12085_amd", "csrc")
MAIN = r"""
#include <stdio.h>
#include <string.h>
#include "apb_plan.h"
int main() {
  char rule[32];
  long long a[8];
  while (scanf("%31s", rule) == 1) {
    if (!strcmp(rule, "attention")) {
      for (int i = 0; i < 6; ++i) if (scanf("%lld", &a[i]) != 1) return 1;
      printf("%d\n", (int)apb::attention_key_split(a[0], a[1], a[2], a[3], a[4], a[5]));
    } else if (!strcmp(rule, "decode")) {
      for (int i = 0; i < 7; ++i) if (scanf("%lld", &a[i]) != 1) return 1;
      const apb::DecodePlan p = apb::plan_decode(a[0], a[1], (int)a[2], a[3], a[4], a[5] != 0, a[6]);
      printf("%d %d %d %d %d %llu\n", p.waves, p.one_launch, p.n_split, p.blocks_per_split,
             p.row_blocks, (unsigned long long)p.workspace_bytes);
    } else if (!strcmp(rule, "gemm")) {
      if (scanf("%lld %lld", &a[0], &a[1]) != 2) return 1;
      const apb::GemmSplit p = apb::gemm_split(a[0], a[1]);
      printf("%d %d\n", p.full, p.nb);
    } else {
      return 1;
    }
  }
  return 0;
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    (d / "plan.cpp").write_text(MAIN)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-I", CSRC, "-o", str(d / "plan"),
                    str(d / "plan.cpp")], check=True)

    def ask(rule, *args):
        out = subprocess.run([str(d / "plan")], input=" ".join([rule, *(str(int(x)) for x in args)]),
                             capture_output=True, text=True, check=True).stdout.split()
        return [int(x) for x in out]

    return ask


def _key_split(plan, n_hosts, host, la, lb, lp, n_q, n_kv, d):
    return plan("attention", la + lb, la, host * lp, lp, n_q, d) == [1]


def test_attention_forms_of_the_gpu_tests(plan):
    one_tile = [(1, 0, 0, 64, 0, 2, 1, 128), (1, 0, 0, 128, 0, 2, 1, 64)]
    for s in attention_forms.SPLIT:
        assert _key_split(plan, *s) == (s not in one_tile), s
    for s in attention_forms.WIDE:
        assert not _key_split(plan, *s), s


@pytest.mark.parametrize("shape, split", [
    # n_hosts, host, La, Lb, l_p, n_q, n_kv, d: row blocks in one round
    ((8, 7, 0, 1024, 1024, 32, 8, 128), True),
    ((8, 7, 0, 1536, 1536, 4, 1, 64), True),
    # more than one round of key-split row blocks: triangles
    ((1, 0, 0, 2048, 0, 32, 8, 128), True),
    ((4, 3, 301, 1023, 127, 32, 8, 128), True),
    ((1, 0, 0, 8192, 0, 8, 2, 64), True),
    ((2, 1, 0, 2048, 2048, 32, 8, 128), True),
    ((8, 7, 256, 1792, 448, 32, 8, 128), True),
    # and row blocks whose keys are nearly all passed on
    ((8, 7, 0, 2048, 2048, 32, 8, 128), False),
    ((8, 7, 0, 1280, 1280, 32, 8, 128), False),
    ((8, 7, 256, 1536, 768, 32, 8, 128), False),
    ((8, 4, 799, 1160, 889, 32, 8, 128), False),
    ((8, 7, 0, 1024, 1024, 40, 8, 128), False),
    ((8, 7, 0, 1024, 1024, 56, 8, 128), False),
    ((4, 3, 0, 8192, 8192, 8, 2, 64), False),
    ((4, 3, 0, 6000, 6000, 8, 2, 64), False),
    ((4, 2, 464, 4056, 3810, 8, 2, 64), False),
    ((3, 2, 134, 1574, 316, 32, 32, 64), False),
    ((3, 2, 386, 4122, 2972, 14, 2, 64), False),
    ((2, 1, 489, 1450, 834, 32, 32, 64), False),
    # the second round has anchor blocks alone
    ((8, 7, 1152, 1024, 1024, 32, 8, 64), False),
    ((8, 7, 1024, 1024, 1024, 32, 8, 128), True),
    # many passed blocks in a tile
    ((16, 15, 50, 500, 20, 32, 8, 128), True),
    ((64, 63, 50, 500, 20, 8, 2, 64), False),
    ((128, 127, 30, 700, 30, 32, 8, 128), False),
    ((26, 25, 0, 1900, 20, 32, 8, 128), False),
    ((17, 16, 0, 1900, 60, 32, 8, 128), True),
    ((26, 25, 0, 1900, 100, 32, 8, 128), True),
    ((26, 25, 0, 600, 100, 4, 1, 64), True),
    ((8, 7, 0, 300, 300, 4, 1, 64), True),
    ((8, 7, 20, 200, 12, 32, 8, 128), True),
    # past one round of 256-row workgroups
    ((1, 0, 0, 2049, 0, 32, 8, 128), False),
    ((1, 0, 0, 1, 0, 257, 257, 128), False),
])
def test_attention_form(plan, shape, split):
    assert _key_split(plan, *shape) == split


NO_LIMIT = 1 << 62


def _decode(plan, n_q, n_kv, d, lc, n_new, app, limit=NO_LIMIT):
    waves, one, n_split, bps, rb, ws = plan("decode", n_q, n_kv, d, lc, n_new, app, limit)
    assert ws == apb.decode_workspace_size(apb.DecodeProblem(n_q, n_kv, d, lc, n_new, app)) \
        or limit != NO_LIMIT
    return ("one launch" if one else waves), n_split, bps


def test_decode_forms_of_the_gpu_tests(plan):
    for s, _ in decode_forms.ONE_LAUNCH:
        blocks = -(-(s[3] + s[4] * s[5]) // 32)
        got = _decode(plan, *s)[0]
        if s == (24, 2, 128, 200, 10, 0):
            assert got == "one launch"  # 120 rows, splits too short for groups
        elif s == (8, 2, 128, 40, 1, 1):
            assert got == 1             # one split
        else:
            assert (got == "one launch") == (blocks <= (12 if s[2] == 128 else 28)), s
    for s, _ in decode_forms.GROUPS:
        assert _decode(plan, *s)[0] == 4, s
    for s, _ in decode_forms.SHORT:
        assert _decode(plan, *s)[0] == 1, s
    assert _decode(plan, 8, 2, 128, 36000, 25, 0)[0] == 4  # its NaN test
    assert [_decode(plan, *s[:6], apb.NOALLOC_SCRATCH_BYTES)[0] for s in no_alloc.CALLS] == \
        [8, 8, 4, "one launch", 1]


@pytest.mark.parametrize("shape, form", [
    # n_q, n_kv, d, Lc, n_new, append: the one-launch form's last length
    ((32, 8, 128, 383, 1, 1), "one launch"),
    ((32, 8, 128, 384, 1, 1), 1),
    ((56, 8, 128, 376, 8, 1), "one launch"),
    ((4, 1, 64, 895, 1, 1), "one launch"),
    ((4, 1, 64, 896, 1, 1), 1),
    ((8, 2, 64, 950, 2, 1), 1),
    # many rows
    ((32, 8, 128, 16384, 32, 1), 8),
    ((32, 8, 128, 16384, 31, 1), 4),
    # three and four row blocks: splits of 8 and 9 blocks of d = 128, 5 and 6 of 64
    ((32, 8, 128, 8150, 24, 1), 1),
    ((32, 8, 128, 8200, 24, 1), 4),
    ((32, 8, 128, 6100, 31, 1), 1),
    ((32, 8, 128, 6150, 31, 1), 4),
    ((8, 2, 64, 20400, 24, 1), 1),
    ((8, 2, 64, 20600, 24, 1), 4),
    ((8, 2, 64, 15300, 31, 1), 1),
    ((8, 2, 64, 15400, 31, 1), 4),
    ((32, 8, 128, 16384, 16, 1), 1),
])
def test_decode_form(plan, shape, form):
    assert _decode(plan, *shape)[0] == form


def test_decode_plan_within_a_limit(plan):
    # one part per split of (d + 1) floats per row; the one-launch form needs the
    # scratch of the splits all the same, and gives way to a single split
    part = 8 * 1 * 129 * 4
    assert _decode(plan, 8, 2, 128, 300, 1, 1, part - 1)[1] == 0
    assert _decode(plan, 8, 2, 128, 300, 1, 1, part) == (1, 1, 10)
    assert _decode(plan, 8, 2, 128, 300, 1, 1, 2 * part) == ("one launch", 1, 10)
    assert _decode(plan, 8, 2, 128, 8000, 1, 1, 3 * part) == (1, 3, 84)


@pytest.mark.parametrize("tokens, features, cut", [
    # tokens, 256-feature tiles; 256-token tiles and the width of the others.  The
    # scorer's shapes of the GPU tests:
    (1, 4, (0, 64)),
    (65, 4, (0, 64)),
    (4096, 4, (0, 64)),
    (4097, 4, (0, 96)),
    (6144, 4, (0, 96)),
    (6145, 4, (0, 128)),
    (8192, 4, (0, 128)),
    (8193, 4, (33, 256)),
    (17001, 4, (0, 96)),
    (18500, 4, (64, 64)),
    (20500, 4, (64, 96)),
    (200, 4, (0, 64)),
    (5000, 4, (0, 96)),
    (9000, 1, (0, 64)),
    # the layer's
    (600, 32, (0, 96)),
    (1000, 32, (0, 128)),
    # whole rounds
    (16384, 4, (64, 256)),
    (2048, 32, (8, 256)),
])
def test_gemm_cut(plan, tokens, features, cut):
    full, nb = plan("gemm", tokens, features)
    got = (full, 32 * nb) if nb < 8 else (-(-tokens // 256), 256)
    assert got == cut
    assert nb == 8 or 256 * full <= tokens
