"""A decode step that packs a token in the launch that attends to it: the packed row at the edges of V units, V blocks
and tiles, in every code width, as one chunk and as several, against the oracle and byte for byte against its cache; the fp16 tokens' slices, the
weights' and the query's operands."""
import numpy as np
import pytest
import torch

import exact_scores
import fp16_slices
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
    bound = fp16_slices.bound(q, k, v) if k.shape[2] <= window else P.TOL  # (longer: some tokens are packed)
    assert (np.abs(out - pair.ref.decode_multi(q)) <= bound).all()


@pytest.mark.parametrize("hq,hk,n_new", [(6, 2, 1), (8, 2, 1), (2, 2, 1), (4, 4, 4)])
@pytest.mark.parametrize("context", fp16_slices.CLOSE_CONTEXTS)
def test_fp16_tokens_keep_weights_of_32_bits(P, hq, hk, n_new, context):
    w, q = fp16_slices.close_scores(hq, hk, n_new, context)
    pair, k, v, _ = P.make_pair(w, max_new_tokens=n_new)
    pair.prefill(k, v)
    out = pair.gpu.skvq_decode_attention_multi(torch.from_numpy(q).to(pair.device)).cpu().numpy()
    ref = pair.ref.decode_multi(q)
    error = np.linalg.norm(out - ref) / np.linalg.norm(ref)
    assert error <= fp16_slices.CLOSE_BOUND, error


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
    # 2- and 4-bit keys of one and two groups meet the query as four FP8 numbers per channel, sixteen tokens a product (that all
    # four enter, as they should, shows in test_scores_are_exact)
    w = synth.Workload("parts", 1, hq, hk, 8 + packed, v_bits, group_size=group, window=8, seed=5 + packed, k_bits=k_bits)
    pair, k, v, q = P.make_pair(w, meta=meta)
    pair.prefill(k, v)
    rng = np.random.default_rng(packed)
    rng = np.random.default_rng(packed)
    one = np.zeros_like(q)
    one[..., packed % 128] = -1.75
    for kind, x in {"normal": q, "wide": q * 10.0 ** rng.uniform(-6, 0.5, q.shape), "one channel": one, "zero": 0 * one,
                    "subnormal": q * 1e-6, "large": q * 30}.items():
        x = x.astype(np.float16)
        out, ref = pair.decode_both(x)
        assert np.abs(out - ref).max() <= P.TOL, kind
    # an infinite channel spoils its own head only
    x = q.copy()
    x[0, -1, 3] = np.inf
    out = pair.gpu.skvq_decode_attention(torch.from_numpy(x).to(pair.device)).cpu().numpy()
    assert np.isnan(out[0, -1]).all()
    assert np.abs(out[0, :-1] - pair.ref.decode(q)[0, :-1]).max(initial=0) <= P.TOL


@pytest.mark.parametrize("meta", ["f32", "e4m3"])
@pytest.mark.parametrize("case", exact_scores.CASES, ids=lambda c: "-".join(map(str, c)))
def test_scores_are_exact(P, case, meta):
    from paper_2405_06219_amd import binding as B
    x = exact_scores.Case(*case)
    gpu = B.SkvqCache(*x.cache_args(), sm_scale=x.sm_scale, k_bits=x.k_bits, meta=meta)
    gpu.skvq_prefill_quantize(torch.from_numpy(x.k).to("cuda:0"), torch.from_numpy(x.v).to("cuda:0"))
    out = gpu.skvq_decode_attention(torch.from_numpy(x.q).to("cuda:0")).cpu().numpy()
    assert np.abs(out - x.oracle(meta)).max() <= exact_scores.BOUND
