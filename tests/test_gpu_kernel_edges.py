"""Edges of the kernels' dispatch rules and tiles, against the oracle (through the C ABI)."""
import numpy as np
import pytest
import torch

import parity_util as P

pytestmark = pytest.mark.gpu

D = 128


def prefill_inputs(B, Hq, Hk, T, seed):
    rng = np.random.default_rng(seed)
    q = rng.standard_normal((B, Hq, T, D)).astype(np.float16)
    k = (rng.standard_normal((B, Hk, T, D)) * 10 ** rng.uniform(-1.0, 1.0, (1, Hk, 1, D))).astype(np.float16)
    v = (rng.standard_normal((B, Hk, T, D)) * 10 ** rng.uniform(-1.0, 1.0, (1, Hk, 1, D))).astype(np.float16)
    return q, k, v


# heads that divide by the eight chiplets (each takes neighbouring heads) and heads that do not, at lengths
# on either side of a query block and of a key tile
@pytest.mark.parametrize("B,Hq,Hk,T", [(1, 8, 2, 513), (1, 16, 16, 255), (2, 12, 3, 257), (1, 7, 7, 256), (1, 1, 1, 65),
                                       (3, 8, 1, 63)])
def test_prefill_attention_grid(B, Hq, Hk, T):
    from oracle import skvq_oracle as O
    from paper_2405_06219_amd import binding as Bd
    print("case", B, Hq, Hk, T, flush=True)
    q, k, v = prefill_inputs(B, Hq, Hk, T, 4100 + T)
    perm = np.tile(np.arange(D, dtype=np.int32), (Hk, 1))
    one = np.ones((Hk, 1), np.float32)
    ref = O.OracleCache(B, Hq, Hk, 128, 1.5, 8, 8, perm, perm, one, one).prefill_attention(q, k, v)
    gpu = Bd.SkvqCache(B, Hq, Hk, 128, 1.5, 8, 8, perm, perm, one, one)
    out = gpu.skvq_prefill_attention(*(torch.from_numpy(x).to("cuda:0") for x in (q, k, v)))
    torch.cuda.synchronize()
    # fp32 accumulation of fp16 products and weights of ~22 bits: 1e-4 was the largest seen on such inputs
    # (|v| up to 40); the library's bound for every attention output is P.TOL = 2e-3
    assert np.abs(out.cpu().numpy() - ref).max() <= P.TOL


# steps that append inside the attention launch with one, two and three chunks per kv head (few workgroups),
# from an empty cache, across a V block's and a tile's edge, and the two-launch form beside it (300 heads)
@pytest.mark.parametrize("batch,heads,context,splits", [(1, 2, 0, 0), (1, 3, 190, 0), (2, 2, 700, 2), (1, 2, 900, 3),
                                                        (75, 4, 140, 0)])
def test_step_of_few_workgroups(batch, heads, context, splits):
    from paper_2405_06219_amd import synth
    print("case", batch, heads, context, splits, flush=True)
    w = synth.Workload("few", batch, heads, heads, context, 2.0 if heads == 3 else 1.5, group_size=64, window=16, seed=9)
    pair, k, v, q = P.make_pair(w, extra_tokens=36)
    if context:
        pair.prefill(k, v)
    if splits:
        pair.gpu.skvq_set_num_splits(splits)
    for s in range(4 if batch > 2 else 36):
        out, ref = pair.append_decode_both(*synth.make_new_token(w, s), q)
        assert np.abs(out - ref).max() <= P.TOL, s
    pair.assert_buffers_equal()


# more than four rows per kv head, few kv heads (workgroups of four rows): 5 .. 16 and 64 rows, every code
# format with one and two groups, packed regions of none, one and a few tokens around a tile's and a V block's
# edge, sinks, one and more chunks
WIDE_CASES = [
    # q heads, kv heads, query tokens, context, batch, K bits, V bits, group, meta, sinks, window, chunks
    (5, 1, 1, 16 + 1, 1, 2.0, 1.5, 128, "f32", 0, 16, 0),
    (8, 1, 2, 16 + 63, 2, 2.0, 1.5, 128, "e4m3", 0, 16, 0),
    (6, 2, 5, 16 + 64, 1, 2.0, 1.5, 64, "f32", 0, 16, 1),
    (8, 2, 2, 16 + 65, 1, 2.0, 2.0, 128, "f16", 0, 16, 0),
    (8, 2, 4, 700, 1, 2.0, 2.0, 64, "e4m3", 5, 32, 3),
    (8, 1, 8, 1100, 1, 2.0, 4.0, 128, "e4m3", 0, 128, 0),
    (4, 1, 4, 33 + 95, 3, 2.0, 4.0, 64, "f16", 0, 33, 0),
    (7, 1, 2, 33 + 97, 1, 3.0, 3.0, 128, "f32", 1, 33, 0),
    (6, 1, 2, 900, 1, 3.0, 3.0, 64, "e4m3", 0, 128, 2),
    (8, 1, 1, 800, 1, 4.0, 1.5, 128, "f16", 0, 128, 4),
    (8, 4, 3, 600, 1, 4.0, 1.5, 64, "f32", 3, 128, 0),
    (5, 1, 3, 520, 1, 4.0, 2.0, 128, "f32", 0, 64, 0),
    (8, 2, 4, 2000, 1, 4.0, 4.0, 64, "e4m3", 5, 128, 5),
    (5, 1, 2, 12, 1, 4.0, 4.0, 128, "f32", 0, 16, 0),   # nothing packed
]

# ... and with more (sequence, kv head) pairs than the compute units have room for at four rows a workgroup
# (decode_wide_kernel, sixteen rows a workgroup): 5 .. 16 rows in one pass, 20 and 24 in two (the second one
# ragged), the same edges and formats
MANY_HEADS = [
    (5, 1, 1, 16 + 1, 140, 2.0, 1.5, 128, "f32", 0, 16, 0),
    (16, 2, 2, 16 + 63, 70, 2.0, 1.5, 128, "e4m3", 0, 16, 0),
    (6, 2, 5, 16 + 64, 70, 2.0, 1.5, 64, "f32", 0, 16, 1),
    (10, 2, 4, 16 + 65, 68, 2.0, 1.5, 128, "f32", 0, 16, 0),     # 20 rows
    (12, 4, 8, 300, 35, 2.0, 1.5, 64, "e4m3", 5, 32, 0),         # 24 rows
    (10, 2, 4, 700, 24, 2.0, 2.0, 128, "f16", 0, 16, 3),         # 20 rows, three chunks
    (6, 2, 8, 16 + 70, 68, 3.0, 3.0, 128, "f32", 1, 16, 0),      # 24 rows
    (8, 2, 4, 700, 24, 2.0, 2.0, 64, "e4m3", 5, 32, 3),
    (4, 1, 4, 33 + 95, 140, 2.0, 4.0, 64, "f16", 0, 33, 0),
    (8, 1, 2, 400, 70, 2.0, 4.0, 128, "e4m3", 0, 128, 2),
    (16, 2, 2, 420, 70, 3.0, 3.0, 64, "e4m3", 0, 64, 0),
    (8, 1, 1, 300, 140, 4.0, 1.5, 128, "f16", 0, 33, 0),
    (8, 4, 8, 600, 35, 4.0, 1.5, 64, "f32", 3, 128, 0),
    (5, 1, 3, 300, 140, 4.0, 2.0, 128, "f32", 0, 64, 0),
    (16, 4, 4, 300, 35, 4.0, 2.0, 64, "f16", 0, 64, 0),
    (8, 2, 4, 900, 24, 4.0, 4.0, 64, "e4m3", 5, 128, 5),
    (5, 1, 2, 12, 140, 4.0, 4.0, 128, "f32", 0, 16, 0),          # nothing packed
]


@pytest.mark.parametrize("case", WIDE_CASES + MANY_HEADS, ids=lambda c: "-".join(map(str, c)))
def test_many_rows_per_kv_head(case):
    from paper_2405_06219_amd import synth
    print("case", case, flush=True)
    hq, hk, n_new, context, batch, k_bits, v_bits, group, meta, sinks, window, splits = case
    w = synth.Workload("rows", batch, hq, hk, context, v_bits, group_size=group, window=window, k_bits=k_bits, seed=31)
    pair, k, v, q1 = P.make_pair(w, extra_tokens=n_new + 6, n_sink=sinks, meta=meta, max_new_tokens=n_new)
    pair.prefill(k, v)
    if splits:
        pair.gpu.skvq_set_num_splits(splits)
    for s in range(n_new):
        pair.append(*synth.make_new_token(w, s))
    q = np.random.default_rng(context).standard_normal((batch, n_new, hq, D)).astype(np.float16)
    qd = torch.from_numpy(q).to(pair.device)
    out = pair.gpu.skvq_decode_attention_multi(qd).cpu().numpy()
    assert np.abs(out - pair.ref.decode_multi(q)).max() <= P.TOL
    wide = "decode_wide_kernel" in decode_kernels(lambda: pair.gpu.skvq_decode_attention_multi(qd))
    assert wide == (case in MANY_HEADS)
    for s in range(4):   # with more than four query heads per kv head: the step's append inside the launch
        out, ref = pair.append_decode_both(*synth.make_new_token(w, 50 + s), q1)
        assert np.abs(out - ref).max() <= P.TOL, s
    pair.assert_buffers_equal()


# the prompt quantizer at every number of tokens of a last sub-block (1 .. 8) and at a V block's edge, for
# every value width, with equal and unequal groups, compact pairs and values down to fp16's subnormals
@pytest.mark.parametrize("packed,k_bits,v_bits,group,meta,bounds", [
    (1, 3.0, 3.0, 64, "e4m3", [0, 32, 128]), (2, 4.0, 4.0, 32, "e4m3", [0, 16, 32, 64, 128]), (3, 2.0, 2.0, 64, "f16", [0, 112, 128]),
    (4, 2.0, 4.0, 64, "f32", None), (5, 4.0, 4.0, 64, "e4m3", None), (6, 3.0, 3.0, 32, "f16", [0, 48, 64, 112, 128]),
    (7, 4.0, 1.5, 32, "e4m3", None), (8, 3.0, 3.0, 128, "f32", None), (31, 3.0, 3.0, 64, "e4m3", [0, 80, 128]),
    (33, 2.0, 2.0, 128, "e4m3", None), (37, 2.0, 1.5, 64, "e4m3", [0, 96, 128]), (35, 4.0, 2.0, 128, "f32", None)])
def test_prompt_quantizer_tails(packed, k_bits, v_bits, group, meta, bounds):
    from paper_2405_06219_amd import synth
    print("case", packed, k_bits, v_bits, group, meta, bounds, flush=True)
    w = synth.Workload("tails", 2, 3, 3, 16 + packed, v_bits, group_size=group, window=16, k_bits=k_bits, seed=packed)
    pair, k, v, _ = P.make_pair(w, meta=meta, group_bounds=bounds)
    k[0, 1, 0] = (k[0, 1, 0].astype(np.float32) * 1e-6).astype(np.float16)    # subnormal
    v[1, 2, packed - 1] = (v[1, 2, packed - 1].astype(np.float32) * 2e-6).astype(np.float16)
    v[0, 0, 0] = -0.0
    pair.prefill(k, v)
    pair.assert_buffers_equal()


# chunks combined by the workgroup that ends last (2 .. 8) and by the second launch (9): one to four rows, a
# partly filled last pass of rows, chunks of one tile, the same counters call after call
@pytest.mark.parametrize("hq,hk,n_new,context,batch,splits", [(2, 2, 1, 128 + 65, 1, 2), (3, 3, 1, 700, 2, 8), (4, 2, 1, 900, 1, 7),
                                                              (6, 2, 1, 640, 2, 3), (8, 2, 1, 700, 1, 8), (4, 1, 1, 800, 3, 9),
                                                              (2, 1, 2, 700, 1, 5), (3, 3, 3, 1000, 1, 8), (4, 4, 1, 2048, 1, 0)])
def test_chunks_combined_in_the_launch(hq, hk, n_new, context, batch, splits):
    from paper_2405_06219_amd import synth
    print("case", hq, hk, n_new, context, batch, splits, flush=True)
    w = synth.Workload("last", batch, hq, hk, context, 1.5, group_size=128, seed=77)
    pair, k, v, _ = P.make_pair(w, extra_tokens=8, max_new_tokens=n_new)
    pair.prefill(k, v)
    pair.gpu.skvq_set_num_splits(splits)
    rng = np.random.default_rng(context)
    for s in range(3):
        q = rng.standard_normal((batch, n_new, hq, D)).astype(np.float16)
        o16 = torch.empty(q.shape, dtype=torch.float16, device=pair.device)
        out = pair.gpu.skvq_decode_attention_multi(torch.from_numpy(q).to(pair.device), out_f16=o16).cpu().numpy()
        assert np.abs(out - pair.ref.decode_multi(q)).max() <= P.TOL, s
        assert np.array_equal(o16.cpu().numpy(), out.astype(np.float16))
        pair.append(*synth.make_new_token(w, s))


def test_chunks_combined_in_the_launch_replayed():
    """A captured call replayed with another query each time, eager calls in between: bit for bit the eager result.
    The workspace holds NaN patterns before each replay, so a partial read before it was written would show."""
    from paper_2405_06219_amd import synth
    w = synth.Workload("replay", 1, 4, 2, 900, 1.5, group_size=128, seed=8)
    pair, k, v, q = P.make_pair(w)
    pair.prefill(k, v)
    pair.gpu.skvq_set_num_splits(6)
    qd = torch.from_numpy(q).to(pair.device)
    out = torch.empty(q.shape, dtype=torch.float32, device=pair.device)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        pair.gpu.skvq_decode_attention(qd, out_f32=out)
    rng = np.random.default_rng(5)
    for _ in range(5):
        new = rng.standard_normal(q.shape).astype(np.float16)
        qd.copy_(torch.from_numpy(new))
        eager = pair.gpu.skvq_decode_attention(qd).cpu().numpy()
        assert np.abs(eager - pair.ref.decode(new)).max() <= P.TOL
        out.zero_()
        pair.gpu.buffers["workspace"].fill_(0xFF)
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(out.cpu().numpy(), eager)


def decode_kernels(call):
    """Names of the library's kernels that the call launches."""
    from torch.profiler import ProfilerActivity, profile
    call()
    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CUDA]) as prof:
        call()
        torch.cuda.synchronize()
    known = ("decode_mfma_kernel", "decode_wide_kernel", "merge_kernel", "append_kernel")
    return [k for e in prof.events() for k in known if k in e.name]


# More than four rows per kv head: workgroups of sixteen rows only where those of four do not find room (short
# caches: 13 us with four rows a workgroup, 26 with sixteen, 8 q / 1 kv x 1000 tokens)
@pytest.mark.parametrize("kind,batch,hq,hk,n_new,context,window,wide", [
    ("decode", 1, 8, 1, 1, 1000, 128, False), ("step", 1, 8, 1, 1, 300, 128, False), ("multi", 1, 8, 2, 4, 4000, 128, False),
    ("decode", 8, 64, 8, 1, 600, 128, False), ("multi", 1, 8, 2, 4, 12, 16, False),
    ("multi", 70, 8, 2, 4, 100, 16, True), ("decode", 140, 8, 1, 1, 300, 16, True), ("step", 140, 8, 1, 1, 300, 16, True)])
def test_rows_per_workgroup(kind, batch, hq, hk, n_new, context, window, wide):
    from paper_2405_06219_amd import synth
    print("case", kind, batch, hq, hk, n_new, context, window, flush=True)
    w = synth.Workload("route", batch, hq, hk, context, 1.5, group_size=128, window=window, seed=6)
    pair, k, v, q = P.make_pair(w, extra_tokens=8, max_new_tokens=n_new)
    pair.prefill(k, v)
    dev = pair.device
    q1, qn = torch.from_numpy(q).to(dev), torch.zeros((batch, n_new, hq, D), dtype=torch.float16, device=dev)
    kn, vn = (torch.from_numpy(x).to(dev) for x in synth.make_new_token(w, 0))
    names = decode_kernels({"decode": lambda: pair.gpu.skvq_decode_attention(q1),
                            "multi": lambda: pair.gpu.skvq_decode_attention_multi(qn),
                            "step": lambda: pair.gpu.skvq_append_decode_attention(kn, vn, q1)}[kind])
    assert ("decode_wide_kernel" in names) == wide and ("decode_mfma_kernel" in names) != wide, names


# The chunks that the library chooses, by the partials found in the workspace (one chunk leaves none): one where
# there is little to share, up to eight combined in the launch, more beyond
@pytest.mark.parametrize("hq,hk,context,window,chunks", [
    (1, 1, 16 + 64 * 9, 16, 1), (4, 4, 128 + 64 * 5, 128, 1), (32, 32, 4 + 64 * 16, 4, 1),      # 1.0 .. 1.3 times as long in more
    (4, 1, 128 + 64 * 3, 128, 3), (1, 1, 128 + 64 * 12, 128, 8), (4, 4, 16 + 64 * 31, 16, 8), (1, 1, 16 + 64 * 160, 16, 10)])
def test_number_of_chunks(hq, hk, context, window, chunks):
    from paper_2405_06219_amd import synth
    print("case", hq, hk, context, window, chunks, flush=True)
    w = synth.Workload("chunks", 1, hq, hk, context, 2.0, group_size=128, window=window, seed=12)
    pair, k, v, q = P.make_pair(w)
    pair.prefill(k, v)
    space = pair.gpu.buffers["workspace"]
    space.fill_(0xFF)
    out, ref = pair.decode_both(q)
    assert np.abs(out - ref).max() <= P.TOL
    part = space.cpu().numpy().view(np.uint32).reshape(hq, -1, D + 4)
    written = (part[:, :, 1] != 0xFFFFFFFF).sum(axis=1)
    assert (written == (chunks if chunks > 1 else 0)).all(), written


# Chunks are combined in the launch up to eight, four rows, and a compute unit for every workgroup
@pytest.mark.parametrize("batch,hq,hk,splits,merge", [(1, 4, 4, 8, False), (1, 4, 4, 9, True), (2, 64, 16, 8, False),
                                                      (8, 32, 32, 2, True), (3, 32, 32, 4, True)])
def test_where_chunks_are_combined(batch, hq, hk, splits, merge):
    from paper_2405_06219_amd import synth
    print("case", batch, hq, hk, splits, flush=True)
    w = synth.Workload("where", batch, hq, hk, 16 + 64 * 9, 1.5, group_size=128, window=16, seed=3)
    pair, k, v, q = P.make_pair(w)
    pair.prefill(k, v)
    pair.gpu.skvq_set_num_splits(splits)
    out, ref = pair.decode_both(q)
    assert np.abs(out - ref).max() <= P.TOL
    qd = torch.from_numpy(q).to(pair.device)
    assert ("merge_kernel" in decode_kernels(lambda: pair.gpu.skvq_decode_attention(qd))) == merge


# Steps and merged chunks of 5 .. 8 query heads per kv head in formats without the sixteen-row kernel (four groups,
# unequal groups): several workgroups per chunk, the append in a launch of its own
@pytest.mark.parametrize("hq,hk,k_bits,v_bits,group,bounds,splits", [
    (8, 1, 2.0, 1.5, 32, None, 4), (6, 1, 4.0, 4.0, 32, None, 0), (10, 2, 2.0, 1.5, 64, [0, 32, 128], 5),
    (7, 1, 3.0, 3.0, 64, [0, 96, 128], 9)])
def test_several_workgroups_per_chunk(hq, hk, k_bits, v_bits, group, bounds, splits):
    from paper_2405_06219_amd import synth
    print("case", hq, hk, k_bits, v_bits, group, bounds, splits, flush=True)
    w = synth.Workload("several", 1, hq, hk, 16 + 64 * 9 + 60, v_bits, group_size=group, window=16, k_bits=k_bits, seed=23)
    pair, k, v, q = P.make_pair(w, extra_tokens=10, meta="e4m3", group_bounds=bounds)
    pair.prefill(k, v)
    pair.gpu.skvq_set_num_splits(splits)
    out, ref = pair.decode_both(q)
    assert np.abs(out - ref).max() <= P.TOL
    for s in range(8):   # across a tile's edge
        out, ref = pair.append_decode_both(*synth.make_new_token(w, s), q)
        assert np.abs(out - ref).max() <= P.TOL, s
    pair.assert_buffers_equal()
    qd = torch.from_numpy(q).to(pair.device)
    names = decode_kernels(lambda: pair.gpu.skvq_decode_attention(qd))
    assert "decode_mfma_kernel" in names and ("merge_kernel" in names) == (splits > 1), names   # (one chunk of ten tiles by itself)


# The append inside the sixteen-row launch where the chunk that appends holds fewer tiles than the others (48 tiles
# a chunk and more), across a V block's and a tile's edge
@pytest.mark.parametrize("k_bits,v_bits,group", [(2.0, 1.5, 128), (4.0, 4.0, 64)])
def test_many_rows_step_with_a_shorter_last_chunk(k_bits, v_bits, group):
    from paper_2405_06219_amd import synth
    print("case", k_bits, v_bits, group, flush=True)
    w = synth.Workload("short", 13, 25, 5, 16 + 64 * 97 - 4, v_bits, group_size=group, window=16, k_bits=k_bits, seed=41)
    pair, k, v, q = P.make_pair(w, extra_tokens=10)
    pair.prefill(k, v)
    pair.gpu.skvq_set_num_splits(2)
    for s in range(6):
        out, ref = pair.append_decode_both(*synth.make_new_token(w, s), q)
        assert np.abs(out - ref).max() <= P.TOL, s
    pair.assert_buffers_equal()
    kn, vn = (torch.from_numpy(x).to(pair.device) for x in synth.make_new_token(w, 0))
    qd = torch.from_numpy(q).to(pair.device)
    names = decode_kernels(lambda: pair.gpu.skvq_append_decode_attention(kn, vn, qd))
    assert "decode_wide_kernel" in names and "append_kernel" not in names, names


# The sixteen-row kernel with scores that peak (its reference moves) while the value scales rise by decades from
# tile to tile (its weights are scaled again), four query tokens
@pytest.mark.parametrize("k_bits,v_bits,group,meta", [(2.0, 1.5, 128, "f32"), (2.0, 2.0, 64, "f32"), (4.0, 4.0, 64, "f16")])
def test_many_rows_peaked_softmax_and_rising_values(k_bits, v_bits, group, meta):
    from paper_2405_06219_amd import synth
    print("case", k_bits, v_bits, group, meta, flush=True)
    n_new = 4
    w = synth.Workload("rise", 33, 8, 2, 16 + 64 * 40, v_bits, group_size=group, window=16, k_bits=k_bits, seed=52)
    k, v = synth.make_kv(w)
    rise = 10.0 ** np.linspace(-4.0, 0.0, w.context)      # per wavefront five tiles: several decades between them
    v = (v / np.abs(v.astype(np.float32)).max() * rise[None, None, :, None]).astype(np.float16)
    pk, pv = synth.make_permutations(w, k, v)
    pair = P.Pair(w, w.context + 8, pk, pv, *synth.make_clip(w), sm_scale=0.3, meta=meta, max_new_tokens=n_new)
    pair.prefill(k, v)
    q = np.random.default_rng(9).standard_normal((w.batch, n_new, 8, D)).astype(np.float16)
    qd = torch.from_numpy(q).to(pair.device)
    out = pair.gpu.skvq_decode_attention_multi(qd).cpu().numpy()
    ref = pair.ref.decode_multi(q)
    assert np.abs(out - ref).max() <= P.TOL
    # and relative to each row, whose weight may lie on tokens of any decade: scores of up to 2^7 in the exp2 domain, sums of
    # 128 products truncated at 2^-23 of the sum, give weights off by up to 128 * 2^-23 * 2^7 * ln 2 = 1.4e-3
    rel = np.linalg.norm(out - ref, axis=-1) / np.linalg.norm(ref, axis=-1)
    print("largest relative error of a row %.2e" % rel.max(), flush=True)
    assert rel.max() <= 1.4e-3
    assert "decode_wide_kernel" in decode_kernels(lambda: pair.gpu.skvq_decode_attention_multi(qd))


def test_fp8_pairs_of_every_fp16_number():
    """Scale and zero in FP8 from every finite fp16 number x: rows of x and zeros (zero = alpha x, or 0; scale = alpha |x| / 3),
    three alphas, by the prompt quantizer and (the last rows) by appends; ties, subnormals, saturation, both zeros."""
    from paper_2405_06219_amd import binding as Bd
    from oracle import skvq_oracle as O
    x = np.arange(1 << 16, dtype=np.uint16).view(np.float16)
    x = x[np.isfinite(x)]
    n, window, tail = len(x), 64, 40
    k = np.zeros((1, 3, n + window, D), np.float16)
    k[:, :, :n, 5] = x
    v = np.zeros_like(k)
    v[:, :, :n, 7] = x[::-1]
    perm = np.tile(np.arange(D, dtype=np.int32), (3, 1))
    clip = np.array([[1.0], [0.95], [0.37]], np.float32)
    ref = O.OracleCache(1, 3, 3, 128, 2.0, window, n, perm, perm, clip, clip, fill=0, meta="e4m3")
    gpu = Bd.SkvqCache(1, 3, 3, 128, 2.0, window, n, perm, perm, clip, clip, fill=0, meta="e4m3")
    T = n + window - tail
    assert ref.prefill(np.ascontiguousarray(k[:, :, :T]), np.ascontiguousarray(v[:, :, :T])) == 0
    gpu.skvq_prefill_quantize(*(torch.from_numpy(np.ascontiguousarray(a[:, :, :T])).to("cuda:0") for a in (k, v)))
    for t in range(T, n + window):
        kn, vn = np.ascontiguousarray(k[:, :, t]), np.ascontiguousarray(v[:, :, t])
        assert ref.append(kn, vn) == 0
        gpu.skvq_quantize_append(torch.from_numpy(kn).to("cuda:0"), torch.from_numpy(vn).to("cuda:0"))
    for name, g, r in zip(("k_codes", "v_codes", "k_meta", "v_meta", "k_win", "v_win"), gpu.host_arrays(), ref.arrays()):
        g, r = np.asarray(g), np.asarray(r)
        if g.dtype.itemsize == 2:
            g, r = g.view(np.uint16), r.view(np.uint16)
        assert np.array_equal(g, r), name


# Partials combined by the merge launch, at the edges of its slices (8), batches (32) and sets of lanes (64): against
# the oracle, and against one chunk (the same fp32 sums in another order: 1e-5 of the largest output, as in the
# parity tests of split counts).  The workspace holds NaNs before each call.  Up to eight partials reach the merge
# launch from more than four rows per kv head (four groups: always several workgroups of four); of one row two are
# combined in the launch, for comparison.
@pytest.mark.parametrize("hq,hk,group,splits", [(8, 1, 32, n) for n in (2, 3, 7, 8, 9)] + [(2, 2, 128, 2)] +
                         [(2, 2, 128, n) for n in (9, 31, 32, 33, 64, 65, 96, 97, 127, 128)])
def test_merge_at_its_edges(hq, hk, group, splits):
    from paper_2405_06219_amd import synth
    print("case", hq, hk, group, splits, flush=True)
    w = synth.Workload("merge", 2, hq, hk, 64 * 128 + 16, 2.0, group_size=group, window=16, seed=33)
    pair, k, v, q = P.make_pair(w, extra_tokens=1)
    pair.prefill(k, v)
    qd, ref, outs = torch.from_numpy(q).cuda(), pair.ref.decode(q), []
    for n in (1, splits):
        pair.gpu.skvq_set_num_splits(n)
        pair.gpu.buffers["workspace"].fill_(0xFF)
        outs.append(pair.gpu.skvq_decode_attention(qd).cpu().numpy())
        assert np.abs(outs[-1] - ref).max() <= P.TOL, n
    assert np.abs(outs[1] - outs[0]).max() <= 1e-5 * max(1.0, np.abs(ref).max())
    names = decode_kernels(lambda: pair.gpu.skvq_decode_attention(qd))
    assert ("merge_kernel" in names) == (hq // hk > 4 or splits > 8), names


# caches so long that the distance from a tile to the last packed token, in bytes of key rows, is past 32 bits: the first
# tile's 64 tokens have keys of a prompt, all others a score that makes their weight exactly zero
@pytest.mark.parametrize("k_bits,group,packed", [(4.0, 128, 2 ** 26 + 6), (4.0, 64, 2 ** 26 + 6), (2.0, 128, 2 ** 27 + 6),
                                                 (2.0, 64, 2 ** 27 + 6)])
def test_caches_past_four_gigabytes_of_keys(k_bits, group, packed):
    from paper_2405_06219_amd import synth
    print("case", k_bits, group, packed, flush=True)
    w = synth.Workload("long", 1, 4, 1, 8 + 64, 1.5, group_size=group, window=8, seed=31, k_bits=k_bits)
    pair, k, v, _ = P.make_pair(w, meta="e4m3")
    pair.prefill(k, v)
    q = np.random.default_rng(31).uniform(0.5, 1.5, (1, 4, 128)).astype(np.float16)
    ref = pair.ref.decode(q)
    gpu = type(pair.gpu)(1, 4, 1, group, 1.5, 8, packed, *pair.gpu._keep[:4], k_bits=k_bits, meta="e4m3", fill=0)
    gpu.buffers["k_meta"][1::2] = 0xD8  # zeros of -16, scales of 0: scores below -150, the prompt has some above 0
    for name, buffer in pair.gpu.buffers.items():  # the prompt's 64 packed tokens and its window
        if name != "workspace":
            gpu.buffers[name][:buffer.numel()] = buffer
    gpu.skvq_set_state(packed + 8)
    out = gpu.skvq_decode_attention(torch.from_numpy(q).to("cuda:0"))
    torch.cuda.synchronize()
    assert np.abs(out.cpu().numpy() - ref).max() <= P.TOL
