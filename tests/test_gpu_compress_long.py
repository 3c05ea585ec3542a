"""GPU parity of the compressor's streaming kernel (local blocks past 16384
rows) against the oracle, bit for bit: the edges of its range and of its
blocks, scores that its sampled bracket of the threshold does not fit (it
misses, or more keys fall inside than are kept), brackets with tied groups at
their ends or scores that differ in their last bits alone, ties and non-numbers
at the threshold, and shares of more rows than one list holds."""
import numpy as np
import pytest

import oracle
from paper_2502_12085_amd import inputs
from gpu_util import host_bits, need_gpu, run_compress, say, upload

pytestmark = pytest.mark.gpu


def _sample(n):
    """The places whose scores the kernel samples."""
    i, part = np.arange(4096, dtype=np.uint64), np.uint64(n // 4096)
    at = (i * np.uint64(0x9e3779b9) % np.uint64(1 << 32)) * part >> np.uint64(32)
    return i * part + i * np.uint64(n % 4096) // np.uint64(4096) + at


def _unsampled(n, rng):
    """High scores everywhere but at the sampled places."""
    s = rng.standard_normal(n).astype(np.float32) + 50
    s[_sample(n)] -= 100
    return s


def _between_ties(n, rng):
    """20000 ones, 1000 scores below them, zeros."""
    s = np.zeros(n, np.float32)
    s[:20000] = 1
    s[20000:21000] = rng.uniform(0.1, 0.9, 1000)
    return rng.permutation(s)


def _one_waves_blocks(n, rng):
    """Scores around the threshold in every 16th block of 256 alone."""
    s = rng.choice(np.array([-1, 2], np.float32), n)
    at = np.arange(n) // 256 % 16 == 3
    s[at] = rng.uniform(0, 1, np.count_nonzero(at))
    return s


def _few_values(n, rng, values, share):
    return rng.choice(np.array(values, np.float32), n, p=share)


CASES = {
    # name: (Lb, l_p, n_kv, scores)
    "reg_edge": (16384, 2048, 2, lambda n, r: r.standard_normal(n)),
    "first": (16385, 2048, 2, lambda n, r: r.standard_normal(n)),
    "odd_heads": (20003, 1, 3, lambda n, r: r.standard_normal(n)),
    "all_rows": (16640, 16640, 1, lambda n, r: r.standard_normal(n)),
    "all_but_one": (33023, 33022, 1, lambda n, r: r.standard_normal(n)),
    "long_lists": (40961, 20000, 8, lambda n, r: r.standard_normal(n)),
    "two_block_chunks": (262145, 30000, 1, lambda n, r: r.standard_normal(n)),
    "ascending": (65537, 8000, 1, lambda n, r: np.arange(n)),
    "all_equal": (30000, 3000, 2, lambda n, r: np.ones(n)),
    "ones_at_threshold": (65536, 8192, 2, lambda n, r: r.zipf(1.5, n)),
    "ties_over_capacity": (65536, 26000, 2,
                           lambda n, r: _few_values(n, r, [0, 1, 2], [.1, .5, .4])),
    "bracket_misses": (50000, 25000, 2, _unsampled),
    "close_scores": (65536, 8192, 2, lambda n, r: 1 + 1e-5 * r.standard_normal(n)),
    "close_scores_half": (32768, 16384, 2, lambda n, r: 1 + 1e-5 * r.standard_normal(n)),
    "closer_scores": (30001, 5000, 2, lambda n, r: -3 - 1e-6 * r.standard_normal(n)),
    "tie_above": (65536, 19990, 1, _between_ties),
    "between_ties": (65536, 20500, 1, _between_ties),
    "tie_below": (65536, 21010, 1, _between_ties),
    "one_waves_blocks": (65536, 32000, 2, _one_waves_blocks),
    "more_than_kept": (400003, 200000, 1, lambda n, r: r.standard_normal(n)),
    "few_rows": (20000, 64, 8, lambda n, r: r.standard_normal(n)),
    "zeros_at_threshold": (20000, 10000, 2,
                           lambda n, r: _few_values(n, r, [-1, -0.0, 0.0, 1], [.3, .3, .2, .2])),
    "just_below_zero": (20000, 6000, 2,
                        lambda n, r: _few_values(n, r, [-1e-45, 0.0, 1], [.5, .2, .3])),
    "nan_at_threshold": (20000, 15000, 2,
                         lambda n, r: _few_values(n, r, [np.nan, -np.inf, 1], [.5, .2, .3])),
    "minus_inf_at_threshold": (20000, 8000, 2,
                               lambda n, r: _few_values(n, r, [np.nan, -np.inf, 1], [.2, .5, .3])),
    "inf_at_threshold": (20000, 5000, 2,
                         lambda n, r: _few_values(n, r, [np.inf, 3, -np.inf], [.4, .4, .2])),
}


@pytest.mark.parametrize("case", CASES)
def test_streaming_selection(case):
    need_gpu()
    lb, lp, n_kv, make = CASES[case]
    rng = np.random.default_rng(7)
    la, d = 5, 64
    say(f"[compress long] {case}: Lb {lb} l_p {lp} heads {n_kv}")
    s = np.stack([np.asarray(make(lb, rng), np.float32) for _ in range(n_kv)])
    inp = dict(scores=s, k=rng.integers(0, 65536, (n_kv, la + lb, d), dtype=np.uint16),
               v=rng.integers(0, 65536, (n_kv, la + lb, d), dtype=np.uint16),
               q=np.zeros((1, 1, 8), np.uint16), k_pass=np.zeros((1, 8), np.uint16),
               v_pass=np.zeros((1, 8), np.uint16))
    dv = upload(inp)
    idx, k, v = run_compress(inputs.Problem(2, 1, la, lb, lp, n_kv, n_kv, d), dv["scores"],
                             dv["k"], dv["v"])
    ridx, rk, rv = oracle.compress_ref(s, inp["k"], inp["v"], lp, la)
    assert np.array_equal(idx.cpu().numpy(), ridx)
    assert np.array_equal(host_bits(k), rk) and np.array_equal(host_bits(v), rv)
