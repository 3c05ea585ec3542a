"""Which form of a kernel the host chooses (``csrc/apb_plan.h``, plain C++): the
forms that the GPU tests' shapes are written for are the ones they run, and the
rules hold where a form that was measured slower would be taken."""
import os
import subprocess

import pytest

import test_gpu_attention_split as attention_forms

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
      for (int i = 0; i < 5; ++i) if (scanf("%lld", &a[i]) != 1) return 1;
      printf("%d\n", (int)apb::attention_key_split(a[0], a[1], a[2], a[3], a[4]));
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
    return plan("attention", la + lb, la, host * lp, n_q, d) == [1]


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
    # past one round of 256-row workgroups
    ((1, 0, 0, 2049, 0, 32, 8, 128), False),
    ((1, 0, 0, 1, 0, 257, 257, 128), False),
])
def test_attention_form(plan, shape, split):
    assert _key_split(plan, *shape) == split
