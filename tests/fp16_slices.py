"""Inputs and bounds for decode calls over fp16 tokens: attention without packed tokens, in 64 bits."""
from __future__ import annotations

import numpy as np

from paper_2405_06219_amd import synth

CLOSE_CONTEXTS = (8, 15, 31)
# Of the outputs' norm, where all tokens weigh about the same and no score's rounding shows.  A rounding is 2^-25.8 in the mean
# square.  An exponential is off by a unit in the last place (2 of these), a slice's eight multiply-adds by that of partial sums that
# grow with random signs (4.5), its scaling and the slices' sum (3), the sum of weights (2), the division (2): sqrt(13.5) of them.
CLOSE_ROUNDING = 2.0 ** -23.9
CLOSE_BOUND = 1.5 * CLOSE_ROUNDING


def close_scores(hq, hk, n_new, context):
    """Workload and queries [8][n_new][hq][D] whose scores are close to one another."""
    w = synth.Workload("weights32", 8, hq, hk, context, 2.0, window=64, seed=78)
    return w, (1e-3 * np.random.default_rng(context).standard_normal((8, n_new, hq, 128))).astype(np.float16)


def attention(q, k, v, weigh=lambda p: p):
    """q [B][n_new][Hq][D] of the last tokens of k, v [B][Hk][T][D]: outputs like q, weights [B][Hq][n_new][T] summing to one, and per
    score sm_scale times the sum of its terms' magnitudes.  weigh: what enters the value sum in the place of exp(score - largest)."""
    q, k, v = (x.astype(np.float64) for x in (q, k, v))
    n_new, T, shared = q.shape[1], k.shape[2], q.shape[2] // k.shape[1]
    k, v, q = np.repeat(k, shared, 1), np.repeat(v, shared, 1), q.transpose(0, 2, 1, 3)
    scale = 1.0 / np.sqrt(q.shape[-1])
    hidden = np.arange(T) > T - n_new + np.arange(n_new)[:, None]
    s = np.where(hidden, -np.inf, scale * (q @ k.swapaxes(2, 3)))
    p = np.exp(s - s.max(-1, keepdims=True))
    out = (weigh(p) @ v) / p.sum(-1, keepdims=True)
    return out.transpose(0, 2, 1, 3), p / p.sum(-1, keepdims=True), scale * (np.abs(q) @ np.abs(k).swapaxes(2, 3))


def bound(q, k, v):
    """Per output.  A score is off by 16 adds that truncate (2^-23) in eight sums at most, and less in the vector arithmetic:
    2^-19 of its terms' magnitudes; a weight by an exponential and its sum: 2^-22.  Both enter the value sum and the sum of weights."""
    _, w, terms = attention(q, k, v)
    v_abs = np.repeat(np.abs(v.astype(np.float64)), q.shape[2] // k.shape[1], 1)
    return 2 * ((w * (2.0 ** -19 * terms + 2.0 ** -22)) @ v_abs).transpose(0, 2, 1, 3)
