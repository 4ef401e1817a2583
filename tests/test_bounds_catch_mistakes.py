"""The bounds of the decode kernels' tests against mistakes planted in 64-bit arithmetic on the same inputs: a bound that such a
mistake passes tests nothing."""
import numpy as np
import pytest

import exact_scores
import fp16_slices
from paper_2405_06219_amd import synth


@pytest.mark.parametrize("case", exact_scores.CASES, ids=lambda c: "-".join(map(str, c)))
def test_every_part_of_the_query_shows(oracle, case):
    x = exact_scores.Case(*case)
    ref, sums = x.oracle()[0], x.part_sums()

    def off(s):
        return np.abs(x.attend(s) - ref).max()
    assert off(sums) <= 2.0 ** -22  # (the oracle's outputs have 24 bits)
    # the sums that the kernel forms are exact in 32 bits: multiples of 2^-20 (parts 1 and 3) and 2^-19 (0 and 2) below 16 and 32
    assert np.abs(sums[1] + sums[3]).max() < 16 and np.abs(sums[0] + sums[2]).max() < 32
    seen = 64 * exact_scores.BOUND
    for part in range(exact_scores.PARTS):
        one = np.arange(exact_scores.PARTS)[:, None, None, None] == part
        assert off(np.where(one, 0, sums)) > seen, ("a part left out", part)
        assert off(np.where(one, 2 * sums, sums)) > seen, ("a part's scale", part)
    # a product that drops what is 2^-14 of its largest term
    largest = np.abs(exact_scores.split(x.reordered_q)[0]).max() * x.codes.max()
    step = 2.0 ** np.ceil(np.log2(largest) - 14)
    coarse = sums.copy()
    coarse[0] = step * np.trunc(sums[0] / step)
    assert off(coarse) > seen or np.array_equal(coarse, sums)
    if x.groups == 2:
        assert off(sums[:, ::-1]) > seen, "groups exchanged"


def rounded(p, bits, to_nearest):
    e = np.floor(np.log2(np.maximum(p, 2.0 ** -100))) + 1 - bits
    return (np.rint if to_nearest else np.trunc)(p * 2.0 ** -e) * 2.0 ** e


@pytest.mark.parametrize("hq,hk,n_new", [(3, 1, 1), (8, 2, 1), (2, 2, 2), (1, 1, 4)])
@pytest.mark.parametrize("context", [4, 7, 8, 9, 17])
def test_weights_of_eleven_bits_show_in_slices(hq, hk, n_new, context):
    w = synth.Workload("slices", 2, hq, hk, context, 2.0, window=64, seed=77)
    k, v = synth.make_kv(w)
    for s in range(6):
        kn, vn = synth.make_new_token(w, s)
        k, v = np.concatenate([k, kn[:, :, None]], 2), np.concatenate([v, vn[:, :, None]], 2)
    q = np.random.default_rng(context).standard_normal((2, n_new, hq, 128)).astype(np.float16)
    exact = fp16_slices.attention(q, k, v)[0]
    wrong = fp16_slices.attention(q, k, v, lambda p: rounded(p, 11, False))[0]
    assert (np.abs(wrong - exact) > fp16_slices.bound(q, k, v)).any()


@pytest.mark.parametrize("hq,hk,n_new", [(6, 2, 1), (8, 2, 1), (2, 2, 1), (4, 4, 4)])
@pytest.mark.parametrize("context", fp16_slices.CLOSE_CONTEXTS)
def test_weights_of_two_fp16_numbers_show(oracle, hq, hk, n_new, context):
    # a weight as two fp16 numbers, four tokens a product, a slice's sums cut off after 24 bits
    w, q = fp16_slices.close_scores(hq, hk, n_new, context)
    k, v = synth.make_kv(w)
    exact, weights, _ = fp16_slices.attention(q, k, v)
    p = weights / weights.max(-1, keepdims=True)
    high = rounded(p, 11, False)
    low = rounded(p - high, 11, True)
    values = np.repeat(v.astype(np.float64), hq // hk, 1)
    wrong = 0
    for first in range(0, context, 8):
        of_slice = np.zeros(p.shape[:3] + (128,))
        for t in range(first, min(first + 8, context), 4):
            for part in (low, high):
                of_slice = of_slice + part[..., t:t + 4] @ values[:, :, t:t + 4]
                of_slice = np.sign(of_slice) * rounded(np.abs(of_slice), 24, False)
        wrong = wrong + of_slice
    wrong = (wrong / p.sum(-1, keepdims=True)).transpose(0, 2, 1, 3)
    error = np.linalg.norm(wrong - exact) / np.linalg.norm(exact)
    assert np.hypot(error, fp16_slices.CLOSE_ROUNDING) > fp16_slices.CLOSE_BOUND  # (the other roundings come on top)
