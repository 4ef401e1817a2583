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
