"""Host-only checks of the C ABI: the library loads, exports what include/skvq.h declares,
and its pure-host entry points (sizes, validation) agree with the oracle and reject bad input."""
import ctypes as C
import os
import re

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
D = 128


@pytest.fixture(scope="module")
def B():
    from paper_2405_06219_amd import binding
    if not os.path.exists(binding.LIB_PATH):
        from paper_2405_06219_amd import build
        build.build()
    return binding


def declared_functions():
    text = open(os.path.join(ROOT, "include", "skvq.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(skvq_[a-z0-9_]+)\s*\(", text)))


def test_library_exports_every_declared_entry_point(B):
    names = declared_functions()
    assert {"skvq_prefill_attention", "skvq_prefill_quantize", "skvq_quantize_append", "skvq_decode_attention", "skvq_create",
            "skvq_destroy", "skvq_sizes"} <= set(names)
    L = B.lib()
    for n in names:
        assert hasattr(L, n), n


def test_missing_library_fails_loudly(B, monkeypatch):
    monkeypatch.setattr(B, "_lib", None)
    monkeypatch.setattr(B, "LIB_PATH", "/nonexistent/libskvq.so")
    with pytest.raises(RuntimeError):
        B.lib()


def cfg_for(B, **kw):
    hk = kw.get("n_kv_heads", 8)
    g = kw.get("group_size", 128)
    perm = kw.pop("perm", np.tile(np.arange(D, dtype=np.int32), (hk, 1)))
    clip = kw.pop("clip", np.ones((hk, D // g), np.float32))
    args = dict(batch=1, n_q_heads=32, n_kv_heads=hk, group_size=g, v_bits=1.5, window=128,
                max_quant_tokens=4096, perm_k=perm, perm_v=perm, clip_k=clip, clip_v=clip)
    args.update(kw)
    return B.make_config(**args)


def test_sizes_agree_with_the_oracle(B, oracle):
    for hk, hq, g, vb, tcap, w, b, sink, meta, kb in [(8, 32, 128, 1.5, 4096, 128, 1, 0, "f32", 2.0),
                                                      (4, 4, 32, 2.0, 1000, 16, 3, 5, "f16", 2.0),
                                                      (2, 16, 64, 1.5, 33, 7, 2, 1, "e4m3", 2.0),
                                                      (8, 32, 64, 4.0, 4097, 128, 1, 5, "e4m3", 4.0),
                                                      (2, 4, 128, 2.0, 65, 9, 2, 0, "f32", 4.0),
                                                      (3, 3, 32, 4.0, 31, 9, 1, 0, "f16", 2.0),
                                                      (8, 32, 64, 3.0, 4097, 128, 1, 5, "e4m3", 3.0)]:
        cfg, keep = cfg_for(B, batch=b, n_q_heads=hq, n_kv_heads=hk, group_size=g, v_bits=vb, window=w,
                            max_quant_tokens=tcap, n_sink=sink, meta=meta, k_bits=kb)
        sizes = B.skvq_sizes(cfg)
        perm = np.tile(np.arange(D, dtype=np.int32), (hk, 1))
        clip = np.ones((hk, D // g), np.float32)
        oc = oracle.OracleCache(b, hq, hk, g, vb, w, tcap, perm, perm, clip, clip, n_sink=sink, meta=meta,
                                k_bits=kb)
        assert sizes[:6] == oc.sizes
        assert sizes[6] == b * hq * (B.SKVQ_MAX_SPLITS + 1) * (D + 4) * 4


def test_validation_rejects_bad_configs(B):
    ok, keep = cfg_for(B)
    assert B.skvq_validate_config(ok) == B.SKVQ_OK
    bad_perm = np.tile(np.arange(D, dtype=np.int32), (8, 1))
    bad_perm[3, 5] = 6                                   # channel 6 twice, 5 missing
    cases = [
        (dict(perm=bad_perm), B.SKVQ_ERR_INVALID_ARG),
        (dict(clip=np.full((8, 1), 1.5, np.float32)), B.SKVQ_ERR_INVALID_ARG),
        (dict(clip=np.full((8, 1), 0.0, np.float32)), B.SKVQ_ERR_INVALID_ARG),
        (dict(clip=np.full((8, 1), np.nan, np.float32)), B.SKVQ_ERR_INVALID_ARG),
        (dict(n_q_heads=30), B.SKVQ_ERR_INVALID_ARG),
        (dict(window=0), B.SKVQ_ERR_INVALID_ARG),
        (dict(n_sink=-1), B.SKVQ_ERR_INVALID_ARG),
        (dict(max_new_tokens=-1), B.SKVQ_ERR_INVALID_ARG),
        (dict(max_new_tokens=65), B.SKVQ_ERR_INVALID_ARG),
        (dict(max_quant_tokens=0), B.SKVQ_ERR_INVALID_ARG),
        (dict(max_quant_tokens=2 ** 31 - 64), B.SKVQ_ERR_UNSUPPORTED),   # packed token numbers are 32-bit in the kernels
        (dict(batch=0), B.SKVQ_ERR_INVALID_ARG),
        (dict(head_dim=64), B.SKVQ_ERR_UNSUPPORTED),
        (dict(group_size=16, clip=np.ones((8, 8), np.float32)), B.SKVQ_ERR_UNSUPPORTED),
        (dict(k_bits=1.5), B.SKVQ_ERR_UNSUPPORTED),
        (dict(k_bits=3.0), B.SKVQ_ERR_UNSUPPORTED),        # 3-bit keys need 3-bit values
        (dict(v_bits=3.0), B.SKVQ_ERR_UNSUPPORTED),
        (dict(n_q_heads=128), B.SKVQ_ERR_UNSUPPORTED),     # 16 query heads per kv head
        # unequal groups: D/G + 1 ascending boundaries from 0 to D, multiples of 16
        (dict(group_size=32, clip=np.ones((8, 4), np.float32), group_bounds=[0, 32, 32, 96, 128]), B.SKVQ_ERR_INVALID_ARG),
        (dict(group_size=32, clip=np.ones((8, 4), np.float32), group_bounds=[16, 32, 64, 96, 128]), B.SKVQ_ERR_INVALID_ARG),
        (dict(group_size=32, clip=np.ones((8, 4), np.float32), group_bounds=[0, 32, 64, 96, 112]), B.SKVQ_ERR_INVALID_ARG),
        (dict(group_size=64, clip=np.ones((8, 2), np.float32), group_bounds=[0, 40, 128]), B.SKVQ_ERR_UNSUPPORTED),
    ]
    for kw, want in cases:
        cfg, keep = cfg_for(B, **kw)
        assert B.skvq_validate_config(cfg) == want, kw
        with pytest.raises(B.SkvqError):
            B.skvq_sizes(cfg)
    largest, keep_l = cfg_for(B, max_quant_tokens=2 ** 31 - 65)
    assert B.skvq_validate_config(largest) == B.SKVQ_OK
    good, keep2 = cfg_for(B, group_size=32, clip=np.ones((8, 4), np.float32), group_bounds=[0, 16, 32, 48, 128])
    uniform, keep3 = cfg_for(B, group_size=32)
    assert B.skvq_validate_config(good) == B.SKVQ_OK and B.skvq_sizes(good) == B.skvq_sizes(uniform)
    # the workspace grows with the number of query tokens per call
    multi, keep4 = cfg_for(B, max_new_tokens=4)
    assert B.skvq_sizes(multi)[6] == 4 * B.skvq_sizes(ok)[6] and B.skvq_sizes(multi)[:6] == B.skvq_sizes(ok)[:6]
    assert B.lib().skvq_validate_config(None) == B.SKVQ_ERR_INVALID_ARG
    # create refuses a bad config and null / misaligned buffers before touching the device
    cfg, keep = cfg_for(B, window=0)
    h = C.c_void_p()
    bufs = B.skvq_buffers(*([16] * 7))
    assert B.lib().skvq_create(C.byref(cfg), C.byref(bufs), C.byref(h)) == B.SKVQ_ERR_INVALID_ARG
    assert B.lib().skvq_create(C.byref(ok), None, C.byref(h)) == B.SKVQ_ERR_INVALID_ARG
    bufs = B.skvq_buffers(*([16] * 6 + [8]))
    assert B.lib().skvq_create(C.byref(ok), C.byref(bufs), C.byref(h)) == B.SKVQ_ERR_INVALID_ARG
    assert not h.value
    # the hot calls refuse a null cache before anything else
    L = B.lib()
    assert L.skvq_quantize_append(None, None, None, None) == B.SKVQ_ERR_INVALID_ARG
    assert L.skvq_decode_attention(None, None, None, None, None) == B.SKVQ_ERR_INVALID_ARG
    assert L.skvq_append_decode_attention(None, None, None, None, None, None, None) == B.SKVQ_ERR_INVALID_ARG
    assert L.skvq_prefill_quantize_filtered(None, None, None, 0, None, None) == B.SKVQ_ERR_INVALID_ARG
    assert L.skvq_prefill_attention_quantize(None, None, None, None, 1, None, None, None) == B.SKVQ_ERR_INVALID_ARG
    assert L.skvq_quantize_append_filtered(None, None, None, 1, None) == B.SKVQ_ERR_INVALID_ARG
    assert B.lib().skvq_status_string(B.SKVQ_ERR_CAPACITY) == b"packed region full"
    B.lib().skvq_destroy(None)


def test_reorder_calibration_equals_the_oracle(B, oracle):
    """skvq_calibrate_reorder is host code: the same permutation and boundaries as the oracle's
    KMeans on the same statistics, for every group size and granularity; bad arguments refused."""
    rng = np.random.default_rng(77)
    for trial in range(12):
        hk = int(rng.integers(1, 5))
        g = int(rng.choice([32, 64, 128]))
        gran = int(rng.choice([1, 16, 32]))
        sc = 10 ** rng.uniform(-1.5, 1.0, (hk, D))
        if trial % 3 == 0:          # a few outlier channels
            sc *= np.where(rng.random((hk, D)) < 0.08, 15.0, 1.0)
        stats = np.stack([-sc * rng.uniform(0.2, 1.0, (hk, D)), sc * rng.uniform(0.2, 1.0, (hk, D))], axis=2).astype(np.float32)
        perm, bounds = B.skvq_calibrate_reorder(stats, g, gran, 100)
        rperm, rbounds = oracle.calibrate_reorder(stats, g, gran, 100)
        assert np.array_equal(perm, rperm) and np.array_equal(bounds, rbounds), (trial, hk, g, gran)
        assert all(sorted(perm[h]) == list(range(D)) for h in range(hk))
        assert np.all(bounds % gran == 0) and np.all(np.diff(bounds, axis=1) >= gran)
    stats = np.zeros((1, D, 2), np.float32)
    with pytest.raises(B.SkvqError):
        B.skvq_calibrate_reorder(stats, 48)
    with pytest.raises(B.SkvqError):
        B.skvq_calibrate_reorder(stats, 32, 24)
    stats[0, 3, 1] = np.inf
    with pytest.raises(B.SkvqError):
        B.skvq_calibrate_reorder(stats, 32)


def test_library_reorder_is_lloyds_kmeans_and_recovers_planted_families(B):
    """The library's own clustering, checked without the oracle: against scikit-learn's Lloyd KMeans
    from the stated start (same partition of the channels), and on planted channel families of
    unequal sizes (clusters = families, listed by range; members by their own range)."""
    from sklearn.cluster import KMeans
    rng = np.random.default_rng(1402)
    for G in (32, 64):
        ng = D // G
        sc = 10 ** rng.uniform(-1.5, 1.0, D)
        stats = np.stack([-sc * rng.uniform(0.3, 1.0, D), sc * rng.uniform(0.3, 1.0, D)], axis=1).astype(np.float32)[None]
        perm, bounds = B.skvq_calibrate_reorder(stats, G, 1, 100)
        f = stats[0].astype(np.float64)
        order = np.lexsort((np.arange(D), f[:, 1] - f[:, 0]))
        init = np.stack([f[order[j * G:(j + 1) * G]].mean(axis=0) for j in range(ng)])
        km = KMeans(n_clusters=ng, init=init, n_init=1, algorithm="lloyd", max_iter=100, tol=0.0).fit(f)
        theirs = {frozenset(np.flatnonzero(km.labels_ == j)) for j in range(ng)}
        ours = {frozenset(perm[0, bounds[0, j]:bounds[0, j + 1]]) for j in range(ng)}
        assert ours == theirs
        # no move of the centres allowed: the clusters are the nearest initial centroids
        perm0, bounds0 = B.skvq_calibrate_reorder(stats, G, 1, 0)
        d2 = ((f[:, None, :] - init[None]) ** 2).sum(axis=2)
        near = d2.argmin(axis=1)
        ours0 = {frozenset(perm0[0, bounds0[0, j]:bounds0[0, j + 1]]) for j in range(ng)} - {frozenset()}
        assert ours0 == {frozenset(np.flatnonzero(near == j)) for j in range(ng)} - {frozenset()}
    sizes, scales = [16, 48, 24, 40], [8.0, 0.05, 1.0, 0.3]
    fam = rng.permutation(np.repeat(np.arange(4), sizes))
    stats = np.zeros((1, D, 2), np.float32)
    for ch in range(D):
        s = scales[fam[ch]] * rng.uniform(0.9, 1.1)
        stats[0, ch] = (-s * rng.uniform(0.8, 1.0), s * rng.uniform(0.8, 1.0))
    perm, bounds = B.skvq_calibrate_reorder(stats, 32, 1, 100)
    by_range = np.argsort(scales)
    assert bounds[0].tolist() == [0] + np.cumsum(np.array(sizes)[by_range]).tolist()
    for j, fj in enumerate(by_range):
        members = perm[0, bounds[0, j]:bounds[0, j + 1]]
        assert set(members) == set(np.flatnonzero(fam == fj))
        assert np.all(np.diff(stats[0, members, 1] - stats[0, members, 0]) >= 0)
    perm16, bounds16 = B.skvq_calibrate_reorder(stats, 32, 16, 100)
    assert np.array_equal(perm16, perm)
    assert np.all(bounds16 % 16 == 0) and np.all(np.diff(bounds16, axis=1) >= 16) and np.all(np.abs(bounds16 - bounds) <= 8)


def test_read_yardstick_refuses_bad_arguments_before_touching_a_device(B):
    """Null pointers, a length that is no multiple of 16 and a misaligned source are refused by the
    host checks (no GPU call is made for them)."""
    L = B.lib()
    L.skvq_read_yardstick.restype = C.c_int
    L.skvq_read_yardstick.argtypes = [C.c_void_p, C.c_size_t, C.c_void_p, C.c_void_p]
    assert L.skvq_read_yardstick(None, 1024, 0x1000, None) == B.SKVQ_ERR_INVALID_ARG
    assert L.skvq_read_yardstick(0x1000, 1024, None, None) == B.SKVQ_ERR_INVALID_ARG
    assert L.skvq_read_yardstick(0x1000, 0, 0x2000, None) == B.SKVQ_ERR_INVALID_ARG
    assert L.skvq_read_yardstick(0x1000, 1000, 0x2000, None) == B.SKVQ_ERR_INVALID_ARG
    assert L.skvq_read_yardstick(0x1008, 1024, 0x2000, None) == B.SKVQ_ERR_INVALID_ARG


def test_read_write_yardstick_refuses_bad_arguments_before_touching_a_device(B):
    """Null pointers, a length that is no multiple of 4096, misaligned buffers and a ratio outside 1..8
    are refused by the host checks (no GPU call is made for them)."""
    L = B.lib()
    L.skvq_read_write_yardstick.restype = C.c_int
    L.skvq_read_write_yardstick.argtypes = [C.c_void_p, C.c_void_p, C.c_size_t, C.c_int32, C.c_void_p]
    bad = B.SKVQ_ERR_INVALID_ARG
    assert L.skvq_read_write_yardstick(None, 0x2000, 4096, 7, None) == bad
    assert L.skvq_read_write_yardstick(0x1000, None, 4096, 7, None) == bad
    assert L.skvq_read_write_yardstick(0x1000, 0x100000, 0, 7, None) == bad
    assert L.skvq_read_write_yardstick(0x1000, 0x100000, 4096 + 16, 7, None) == bad
    assert L.skvq_read_write_yardstick(0x1008, 0x100000, 4096, 7, None) == bad
    assert L.skvq_read_write_yardstick(0x1000, 0x100008, 4096, 7, None) == bad
    assert L.skvq_read_write_yardstick(0x1000, 0x100000, 4096, 0, None) == bad
    assert L.skvq_read_write_yardstick(0x1000, 0x100000, 4096, 9, None) == bad


# The structures that the decode kernels keep in LDS: what is read or written 16 bytes at a time starts at a multiple of
# 16 bytes, in every wavefront's copy.  Layouts are the compiler's own (its host pass), for every rows, table and groups.
def test_lds_vectors_are_aligned(tmp_path):
    import subprocess

    from paper_2405_06219_amd import build

    source = tmp_path / "lds_layout.hip"
    source.write_text("""
#include "skvq_decode_mfma_kernel.h"
#include "skvq_decode_wide_kernel.h"
#include <cstdio>
using namespace skvq;
#define AT(S, M) printf("%zu " #S "::" #M "\\n", __builtin_offsetof(S, M))
template <int R, bool TERNARY, int NG> void narrow() {
  typedef Smem<R, TERNARY, NG> S;
  printf("# rows %d table %d groups %d\\n", R, (int)TERNARY, NG);
  for (int w = 0; w < kNW; ++w) printf("%zu S::wb[%d]\\n", __builtin_offsetof(S, wb) + w * sizeof(typename S::WaveBuf), w);
  AT(S, lut); AT(S, qraw); AT(S, qa); AT(S, qpart); AT(S, qtotal); AT(S, wm); AT(S, wl); AT(S, wz);
}
template <bool TERNARY, int NG> void wide() {
  typedef WideSmem<TERNARY, NG> S;
  printf("# sixteen rows, table %d groups %d\\n", (int)TERNARY, NG);
  AT(S, lut); AT(S, stage); AT(S, ktok); AT(S, vtok); AT(S, qa); AT(S, qraw); AT(S, qpart); AT(S, wm); AT(S, wl); AT(S, wz);
}
template <int R> void rows() {
  narrow<R, true, 1>(); narrow<R, true, 2>(); narrow<R, true, 4>();
  narrow<R, false, 1>(); narrow<R, false, 2>(); narrow<R, false, 4>();
}
int main() {
  rows<1>(); rows<2>(); rows<4>();
  wide<true, 1>(); wide<true, 2>(); wide<false, 1>(); wide<false, 2>();
}
""")
    program = str(tmp_path / "lds_layout")
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    subprocess.run([hipcc, *build.COMMON, "--offload-host-only", str(source), "-o", program], check=True)
    lines = subprocess.run([program], check=True, capture_output=True, text=True).stdout.splitlines()
    assert len(lines) == 18 * 17 + 4 * 11
    where = ""
    for line in lines:
        if line.startswith("#"):
            where = line
        else:
            assert int(line.split()[0]) % 16 == 0, f"{where}: {line}"
