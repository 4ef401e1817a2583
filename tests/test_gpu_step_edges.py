"""A decode step that packs a token in the launch that attends to it: the packed row at the edges of V units, V blocks
and tiles, in every code width, as one chunk and as several, against the oracle and byte for byte against its cache."""
import numpy as np
import pytest
import torch

from paper_2405_06219_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import parity_util
    return parity_util


@pytest.mark.parametrize("hq,hk", [(2, 2), (8, 2)])
@pytest.mark.parametrize("k_bits,v_bits,group,meta", [(2.0, 1.5, 128, "f32"), (2.0, 2.0, 64, "f16"), (3.0, 3.0, 64, "e4m3"),
                                                      (4.0, 4.0, 32, "e4m3"), (4.0, 1.5, 64, "f32")])
@pytest.mark.parametrize("packed,splits", [(0, 1), (7, 1), (31, 1), (63, 1), (127, 2), (520, 8)])
def test_packed_row_at_the_edges(P, hq, hk, k_bits, v_bits, group, meta, packed, splits):
    # packed rows before the first of the steps; 0: the first packed token of all, the window just full
    w = synth.Workload("edges", 1, hq, hk, 16 + packed, v_bits, group_size=group, window=16, seed=21, k_bits=k_bits)
    pair, k, v, q = P.make_pair(w, extra_tokens=4, meta=meta)
    pair.prefill(k, v)
    pair.gpu.skvq_set_num_splits(splits)
    for s in range(3):
        out, ref = pair.append_decode_both(*synth.make_new_token(w, s), q)
        assert np.abs(out - ref).max() <= P.TOL, s
        pair.assert_buffers_equal()


@pytest.mark.parametrize("hq,hk,n_new", [(3, 1, 1), (8, 2, 1), (2, 2, 2), (1, 1, 4)])
@pytest.mark.parametrize("context,window,sinks", [(4, 64, 0), (7, 64, 0), (8, 64, 0), (9, 64, 0), (17, 64, 0), (64, 64, 0), (200, 200, 0),
                                                  (75, 16, 5), (40, 9, 1)])
def test_fp16_tokens_in_slices(P, hq, hk, n_new, context, window, sinks):
    # three and four rows take the fp16 tokens eight at a time through the matrix cores, two rows four at a time
    w = synth.Workload("slices", 2, hq, hk, context, 2.0, window=window, seed=77)
    pair, k, v, _ = P.make_pair(w, extra_tokens=16, n_sink=sinks, max_new_tokens=n_new)
    pair.prefill(k, v)
    pair.gpu.skvq_set_num_splits(1)
    for s in range(6):  # (the ring's oldest row is not its first one afterwards)
        kn, vn = synth.make_new_token(w, s)
        pair.append(kn, vn)
        k, v = np.concatenate([k, kn[:, :, None]], 2), np.concatenate([v, vn[:, :, None]], 2)
    q = np.random.default_rng(context).standard_normal((2, n_new, hq, 128)).astype(np.float16)
    out = pair.gpu.skvq_decode_attention_multi(torch.from_numpy(q).to(pair.device)).cpu().numpy()
    # a score of 128 products summed in 32 bits (base-2 exponent: times 1.45) shifts a weight by as much, and a weight's
    # two fp16 parts keep 22 bits; both once in the sum of weights and once in the outputs
    kq = np.repeat(np.abs(k.astype(np.float64)), hq // hk, 1)
    score = 1.45 * (np.abs(q.astype(np.float64)).transpose(0, 2, 1, 3) @ kq.transpose(0, 1, 3, 2)).max() / np.sqrt(128.0)
    bound = 2 * (136 * 2.0 ** -24 * score + 2.0 ** -21) * np.abs(v.astype(np.float64)).max()
    assert np.abs(out - pair.ref.decode_multi(q)).max() <= bound


@pytest.mark.parametrize("hq,hk,n_new", [(6, 2, 1), (8, 2, 1), (2, 2, 1), (4, 4, 4)])
@pytest.mark.parametrize("context", [8, 15, 31])
def test_fp16_tokens_keep_weights_of_32_bits(P, hq, hk, n_new, context):
    # scores close to one another, so that all tokens weigh about the same and no score's rounding shows
    w = synth.Workload("weights32", 8, hq, hk, context, 2.0, window=64, seed=78)
    pair, k, v, _ = P.make_pair(w, max_new_tokens=n_new)
    pair.prefill(k, v)
    q = (1e-3 * np.random.default_rng(context).standard_normal((8, n_new, hq, 128))).astype(np.float16)
    out = pair.gpu.skvq_decode_attention_multi(torch.from_numpy(q).to(pair.device)).cpu().numpy()
    ref = pair.ref.decode_multi(q)
    # per number: an exponential (a unit in the last place), a multiply-add per token, the sum of weights, a division; each
    # rounds by 2^-25.8 in the mean square, the tokens' values have random signs: sqrt(2 + 5 + 2 + 1) of these are 2^-24.1.
    # A weight in two fp16 numbers is off by up to 2^-22, 2^-22.8 in the mean square where it is full
    assert np.linalg.norm(out - ref) <= 2.0 ** -23 * np.linalg.norm(ref)


@pytest.mark.parametrize("hq,hk", [(1, 1), (2, 1), (4, 1), (7, 1)])
@pytest.mark.parametrize("group,bounds", [(128, None), (64, None), (32, None), (64, (0, 32, 128)), (32, (0, 16, 32, 64, 128))])
@pytest.mark.parametrize("packed", [1, 40, 65])
def test_weights_of_every_row_and_group_count(P, hq, hk, group, bounds, packed):
    # the weights' columns in LDS: 2, 4 or 8 per group, in one operand of sixteen or two
    w = synth.Workload("weights", 1, hq, hk, 8 + packed, 1.5, group_size=group, window=8, seed=9)
    pair, k, v, q = P.make_pair(w, group_bounds=bounds)
    pair.prefill(k, v)
    out, ref = pair.decode_both(q)
    assert np.abs(out - ref).max() <= P.TOL


@pytest.mark.parametrize("hq,hk", [(1, 1), (4, 2), (3, 1), (4, 1)])
@pytest.mark.parametrize("k_bits,group,v_bits,meta", [(2.0, 128, 1.5, "f32"), (2.0, 64, 2.0, "e4m3"), (4.0, 128, 4.0, "f32"),
                                                      (4.0, 64, 1.5, "e4m3")])
@pytest.mark.parametrize("packed", [1, 15, 16, 17, 48, 63, 64, 65, 130])
def test_keys_against_queries_in_parts(P, hq, hk, k_bits, group, v_bits, meta, packed):
    # 2- and 4-bit keys of one and two groups meet the query as four FP8 numbers per channel, sixteen tokens a product
    w = synth.Workload("parts", 1, hq, hk, 8 + packed, v_bits, group_size=group, window=8, seed=5 + packed, k_bits=k_bits)
    pair, k, v, q = P.make_pair(w, meta=meta)
    pair.prefill(k, v)
    rng = np.random.default_rng(packed)
    k_top, v_top = np.abs(k.astype(np.float64)).max(), np.abs(v.astype(np.float64)).max()
    one = np.zeros_like(q)
    one[..., packed % 128] = -1.75
    for kind, x in {"normal": q, "wide": q * 10.0 ** rng.uniform(-6, 0.5, q.shape), "one channel": one, "zero": 0 * one,
                    "subnormal": q * 1e-6, "large": q * 30}.items():
        x = x.astype(np.float16)
        out, ref = pair.decode_both(x)
        # a score of 128 products summed in 32 bits, of a query that its parts miss by 2^-25 of its largest channel at most;
        # values by weights of 22 bits, summed with codes that start six bits below the accumulator's first
        a = np.abs(x.astype(np.float64))
        score = 1.45 / np.sqrt(128.0) * k_top * (136 * 2.0 ** -24 * a.sum(-1).max() + 128 * 2.0 ** -25 * a.max())
        assert np.abs(out - ref).max() <= 2 * (score + 2.0 ** -18) * v_top, kind
    # an infinite channel spoils its own head only
    x = q.copy()
    x[0, -1, 3] = np.inf
    out = pair.gpu.skvq_decode_attention(torch.from_numpy(x).to(pair.device)).cpu().numpy()
    assert np.isnan(out[0, -1]).all()
    assert np.abs(out[0, :-1] - pair.ref.decode(q)[0, :-1]).max(initial=0) <= P.TOL
