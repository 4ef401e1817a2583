"""Inputs whose scores are exact in 32 bits only if every step of the score product is: the query as four FP8 (E4M3) numbers
per channel, products that add their 128 terms exactly, scales and groups as they should be.

All query channels are multiples of 2^-20 below 8 (2 with 4-bit codes) or the same times a power of two, most of them in triples x,
y - x, -y under one code, so that a token's score is a few units of 2^-20 left over from terms of up to the largest channel times the
largest code; the parts of a triple round differently and cancel only together.  sm_scale makes a unit 1/4 (2-bit codes) or 1/16
(4-bit codes) of a score.  The groups' scales are 1 and 2, their zeros 0."""
from __future__ import annotations

import numpy as np

from oracle import skvq_oracle as O

D, WINDOW, UNIT = 128, 8, 2.0 ** -20
PARTS, PART_BITS = 4, 5
# The scores' products are exact; the factor sm_scale * log2(e), the exponential and the weights' sums are rounded: a score of up to
# 32 in base 2 twice by 2^-24 of itself, a weight in 22 bits: of a value of 2, once in the outputs and once in the
# sum of weights.
BOUND = 2 * (64 * 2.0 ** -24 + 2.0 ** -22) * 2


class Case:
    """k, v: the packed tokens and a window of zero keys; q [1][heads][D]; 2^shift: the size of the query."""

    def __init__(self, k_bits, groups, heads, packed, shift=0, seed=0):
        rng = np.random.default_rng([seed, int(k_bits), groups, heads, packed])
        self.k_bits, self.groups, self.heads = k_bits, groups, heads
        levels, size, top = int(2 ** k_bits), D // groups, 2 if k_bits == 2.0 else 0  # largest channel in [2^top, 2^(top + 1))
        self.step = 4 if k_bits == 2.0 else 16
        self.sm_scale = 2.0 ** -shift / UNIT / self.step
        q, k = np.zeros((heads, D)), np.zeros((packed, D))  # in reordered order
        for g in range(groups):
            k[:, g * size + 1] = levels - 1  # (codes 0 and levels - 1 in every group)
            q[:, g * size + 2:g * size + 10] = UNIT * rng.choice([1, 1, -1], (heads, 8))
            k[:, g * size + 2:g * size + 10] = rng.integers(0, levels, (packed, 8))
            for n, p in enumerate(range(g * size + 10, (g + 1) * size - 2, 3)):
                e = top if n == 0 else rng.integers(-10, top)
                x = rng.integers(1024, 2048, heads)
                y = (rng.random(heads) * x).astype(np.int64)
                q[:, p:p + 3] = np.stack([x, y - x, -y], 1) * rng.choice([-1, 1], (heads, 1)) * 2.0 ** (e - 10)
                k[:, p:p + 3] = rng.integers(0, levels, (packed, 1))
        self.perm = rng.permutation(D).astype(np.int32)[None]
        order = np.argsort(self.perm[0])
        self.reordered_q, self.codes, self.scales = q, k, 1.0 + np.arange(groups)
        self.q = np.ascontiguousarray((q * 2.0 ** shift)[:, order][None], np.float16)
        assert np.array_equal(self.q[0].astype(np.float64), (q * 2.0 ** shift)[:, order])
        T = packed + WINDOW
        self.k, self.v = np.zeros((1, 1, T, D), np.float16), rng.integers(0, 3, (1, 1, T, D)).astype(np.float16)
        self.k[0, 0, :packed] = (k * np.repeat(self.scales, size))[:, order]
        self.v[..., 0], self.v[..., 1], self.v[..., D // 2], self.v[..., D // 2 + 1] = 0, 2, 0, 2  # (scale 1, zero 0)

    def cache_args(self):
        """Of OracleCache and SkvqCache: kv head, group size, 1.5-bit values, window, room, permutations, clip scales."""
        one = np.ones((1, self.groups), np.float32)
        identity = np.arange(D, dtype=np.int32)[None]
        return (1, self.heads, 1, D // self.groups, 1.5, WINDOW, self.k.shape[2] - WINDOW, self.perm, identity, one, one)

    def oracle(self, meta="f32"):
        ref = O.OracleCache(*self.cache_args(), sm_scale=self.sm_scale, k_bits=self.k_bits, meta=meta)
        assert ref.prefill(self.k, self.v) == 0
        return ref.decode(self.q)

    def attend(self, sums):
        """The attention with these part_sums; the window's scores are zero."""
        scores = np.einsum("pght,g->ht", sums, self.scales)
        s = np.concatenate([scores / UNIT / self.step, np.zeros((self.heads, WINDOW))], 1)
        w = np.exp(s - s.max(1, keepdims=True))
        return (w / w.sum(1, keepdims=True)) @ self.v[0, 0].astype(np.float64)

    def part_sums(self, parts=PARTS):
        """Per part the products' sums [part][group][head][token]."""
        return np.stack([[p[:, s] @ self.codes[:, s].T for s in (slice(g * D // self.groups, (g + 1) * D // self.groups)
                                                                 for g in range(self.groups))] for p in split(self.reordered_q)[:parts]])


def e4m3(x):
    """Rounded to FP8 E4M3, ties to even (below its largest number)."""
    e = np.maximum(np.floor(np.log2(np.maximum(np.abs(x), 2.0 ** -30))), -6)
    return np.rint(x * 2.0 ** (3 - e)) * 2.0 ** (e - 3)


def split(q):
    """The query as a sum of four arrays, each a multiple of 2^-(9 + 5 part)."""
    parts, rest = [], q.astype(np.float64)
    for part in range(PARTS):
        p = e4m3(rest * 2.0 ** (PART_BITS * part)) * 2.0 ** -(PART_BITS * part)
        parts.append(p)
        rest = rest - p
    return parts


CASES = [(k_bits, groups, heads, packed, shift) for k_bits in (2.0, 4.0) for groups in (1, 2) for heads in (1, 2, 3, 4)
         for packed, shift in ((3, 0), (17, 5), (64, -2), (130, 0))]
