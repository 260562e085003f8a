"""Host-side checks of the C ABI (no GPU): the library loads, exports every declared symbol,
and rejects bad arguments before anything is launched."""
import ctypes
import os
import re
import subprocess
import sys

import pytest

import paper_2503_02236_amd as vq
from paper_2503_02236_amd.binding import SYMBOLS, vq_kv_t, vq_weight_t

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "include", "vq_mi355x.h")

VQ_ERR_NULL, VQ_ERR_SHAPE, VQ_ERR_UNSUPPORTED, VQ_ERR_ALIGN, VQ_ERR_WORKSPACE = -1, -2, -3, -4, -5
P = 0x10000  # a 16-byte aligned fake device address; never dereferenced on the error paths


def declared_functions():
    text = open(HEADER).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(vq_[a-z_]+)\s*\(", text)))


def test_header_declares_and_library_exports_the_same_symbols():
    names = declared_functions()
    assert {"vq_gemv", "vq_gemm", "vq_attn_decode", "vq_dequant", "vq_kv_dequant"} <= set(names)
    lib = vq.lib()
    for n in names:
        assert hasattr(lib, n), n
    assert sorted(SYMBOLS) == names       # the binding wraps exactly what the header declares


def test_status_strings():
    assert vq.status_str(0) == "VQ_OK"
    for s in range(-6, 0):
        assert vq.status_str(s).startswith("VQ_ERR_")
    assert "unknown" in vq.status_str(-99)
    assert vq.lib().vq_version() >= 100


def weight(**kw):
    d = dict(N=64, K=64, v=8, code_bits=8, n_codebooks=1, n_entries=256, codes=P, codebooks=P, scale=None,
             gemv_pack=None)
    d.update(kw)
    return vq_weight_t(**d)


def kvdesc(**kw):
    d = dict(B=1, H=1, D=128, T=16, v=4, n_entries=256, cb_groups=1, k_codes=P, v_codes=P, k_codebooks=P,
             v_codebooks=P, seq_lens=None)
    d.update(kw)
    return vq_kv_t(**d)


def gemv(w, x=P, bs=1, y=P, ws=None, ws_bytes=0):
    return vq.lib().vq_gemv(ctypes.byref(w), x, bs, y, ws, ws_bytes, None)


def gemm(w, x=P, M=1, y=P):
    return vq.lib().vq_gemm(ctypes.byref(w), x, M, y, None, 0, None)


@pytest.mark.parametrize("w,want", [
    (weight(codes=None), VQ_ERR_NULL),
    (weight(codebooks=None), VQ_ERR_NULL),
    (weight(v=3), VQ_ERR_UNSUPPORTED),
    (weight(v=16), VQ_ERR_UNSUPPORTED),
    (weight(code_bits=10), VQ_ERR_UNSUPPORTED),
    (weight(n_codebooks=0), VQ_ERR_UNSUPPORTED),
    (weight(n_codebooks=5), VQ_ERR_UNSUPPORTED),
    (weight(n_entries=257), VQ_ERR_UNSUPPORTED),
    (weight(n_entries=0), VQ_ERR_UNSUPPORTED),
    (weight(K=60), VQ_ERR_SHAPE),
    (weight(N=-1), VQ_ERR_SHAPE),
    (weight(codes=P + 8), VQ_ERR_ALIGN),
    (weight(codebooks=P + 2), VQ_ERR_ALIGN),
    (weight(scale=P + 4), VQ_ERR_ALIGN),
])
def test_weight_descriptor_validation(w, want):
    assert gemv(w) == want
    assert gemm(w) == want
    assert vq.lib().vq_dequant(ctypes.byref(w), P, 1, None) == want
    assert vq.lib().vq_gemv_workspace(ctypes.byref(w), 1) == 0


def test_gemv_gemm_argument_validation():
    w = weight()
    assert vq.lib().vq_gemv(None, P, 1, P, None, 0, None) == VQ_ERR_NULL
    assert gemv(w, x=None) == VQ_ERR_NULL
    assert gemv(w, y=None) == VQ_ERR_NULL
    assert gemv(w, bs=0) == VQ_ERR_SHAPE
    assert gemv(w, bs=17) == VQ_ERR_SHAPE
    assert gemv(w, x=P + 2) == VQ_ERR_ALIGN
    assert gemv(w, y=P + 6) == VQ_ERR_ALIGN
    assert gemm(w, M=0) == VQ_ERR_SHAPE
    assert gemm(w, x=None) == VQ_ERR_NULL
    assert gemm(w, y=P + 2) == VQ_ERR_ALIGN
    assert vq.lib().vq_dequant(ctypes.byref(w), None, 1, None) == VQ_ERR_NULL
    # N == 0 is a valid empty problem: success without a launch
    assert gemv(weight(N=0)) == 0
    assert gemm(weight(N=0)) == 0


@pytest.mark.parametrize("kv,want", [
    (kvdesc(k_codes=None), VQ_ERR_NULL),
    (kvdesc(v_codebooks=None), VQ_ERR_NULL),
    (kvdesc(v=3), VQ_ERR_UNSUPPORTED),
    (kvdesc(n_entries=512), VQ_ERR_UNSUPPORTED),
    (kvdesc(D=126), VQ_ERR_SHAPE),
    (kvdesc(cb_groups=3), VQ_ERR_SHAPE),
    (kvdesc(cb_groups=0), VQ_ERR_SHAPE),
    (kvdesc(T=-1), VQ_ERR_SHAPE),
    (kvdesc(k_codes=P + 1), VQ_ERR_ALIGN),
    (kvdesc(seq_lens=P + 2), VQ_ERR_ALIGN),
])
def test_kv_descriptor_validation(kv, want):
    lib = vq.lib()
    assert lib.vq_attn_decode(ctypes.byref(kv), P, 0.1, P, None, 0, None) == want
    assert lib.vq_kv_dequant(ctypes.byref(kv), 0, P, None) == want
    assert lib.vq_attn_decode_workspace(ctypes.byref(kv)) == 0


def test_attention_argument_validation():
    lib = vq.lib()
    kv = kvdesc()
    assert lib.vq_attn_decode(ctypes.byref(kv), None, 0.1, P, None, 0, None) == VQ_ERR_NULL
    assert lib.vq_attn_decode(ctypes.byref(kv), P, 0.1, P + 8, None, 0, None) == VQ_ERR_ALIGN
    assert lib.vq_kv_dequant(ctypes.byref(kv), 2, P, None) == VQ_ERR_SHAPE
    big = kvdesc(T=100000, B=2, H=2)
    need = lib.vq_attn_decode_workspace(ctypes.byref(big))
    assert need > 0                                    # long caches are split and need partials
    assert lib.vq_attn_decode(ctypes.byref(big), P, 0.1, P, None, 0, None) == VQ_ERR_WORKSPACE
    assert lib.vq_attn_decode(ctypes.byref(big), P, 0.1, P, P, need - 1, None) == VQ_ERR_WORKSPACE
    assert lib.vq_attn_decode(ctypes.byref(kvdesc(B=0)), P, 0.1, P, None, 0, None) == 0


def test_attention_channel_parallel_argument_validation():
    lib = vq.lib()
    f, wsq = lib.vq_attn_decode_channel_parallel, lib.vq_attn_decode_channel_parallel_workspace
    cq = kvdesc(cb_groups=32)                            # D = 128, v = 4: 4 channel groups of 8 codebooks
    need = wsq(ctypes.byref(cq))
    assert need == cq.B * cq.H * (128 // 32 + 1) * cq.T * 4
    assert f(ctypes.byref(cq), None, 0.1, P, P, need, None) == VQ_ERR_NULL
    assert f(ctypes.byref(cq), P, 0.1, P + 8, P, need, None) == VQ_ERR_ALIGN
    assert f(ctypes.byref(cq), P, 0.1, P, None, 0, None) == VQ_ERR_WORKSPACE
    assert f(ctypes.byref(cq), P, 0.1, P, P, need - 1, None) == VQ_ERR_WORKSPACE
    assert f(ctypes.byref(cq), P, 0.1, P, P + 4, need, None) == VQ_ERR_ALIGN
    one = kvdesc()                                       # one codebook per head: does not divide over 4 channel groups
    assert wsq(ctypes.byref(one)) == 0
    assert f(ctypes.byref(one), P, 0.1, P, P, 1 << 30, None) == VQ_ERR_UNSUPPORTED
    assert f(ctypes.byref(kvdesc(cb_groups=32, B=0)), P, 0.1, P, None, 0, None) == 0


def test_kv_quantize_argument_validation():
    lib = vq.lib()
    kv = kvdesc()
    f = lib.vq_kv_quantize
    assert f(ctypes.byref(kv), None, P, 1, 0, None) == VQ_ERR_NULL
    assert f(ctypes.byref(kv), P, P + 2, 1, 0, None) == VQ_ERR_ALIGN
    assert f(ctypes.byref(kv), P, P, -1, 0, None) == VQ_ERR_SHAPE
    assert f(ctypes.byref(kv), P, P, 1, -1, None) == VQ_ERR_SHAPE
    assert f(ctypes.byref(kv), P, P, 2, kv.T - 1, None) == VQ_ERR_SHAPE     # runs past the end of the cache
    assert f(ctypes.byref(kv), P, P, 0, 0, None) == 0                       # nothing to do
    assert f(ctypes.byref(kvdesc(v=3)), P, P, 1, 0, None) == VQ_ERR_UNSUPPORTED


def test_packed_gemv_validation():
    import numpy as np
    from paper_2503_02236_amd import workloads as wl
    from paper_2503_02236_amd.binding import vq_gemv_pack_t
    lib = vq.lib()
    w = wl.make_weight(128, 512, 8, 16, 1, 65536, 0.02, seed=9)
    buf, pack = vq.vq_gemv_prepack(w)
    d = weight(N=128, K=512, code_bits=16, n_entries=65536, codes=None)
    assert gemv(d) == VQ_ERR_NULL                                  # neither codes nor a pack
    pack.data = P                                                  # pretend it was uploaded
    d.gemv_pack = ctypes.pointer(pack)
    need = lib.vq_gemv_workspace(ctypes.byref(d), 1)
    assert need == pack.S * 128 * 4 + 4096      # S x N partial sums in blocks of 64 rows, plus one 4 KiB fetch unit
    assert gemv(d) == VQ_ERR_WORKSPACE
    assert gemv(d, ws=P, ws_bytes=need - 1) == VQ_ERR_WORKSPACE
    assert gemv(d, bs=2) == VQ_ERR_NULL                            # bs > 1 needs the canonical codes
    other = weight(N=256, K=512, code_bits=16, n_entries=65536, codes=None)
    other.gemv_pack = ctypes.pointer(pack)
    assert gemv(other, ws=P, ws_bytes=1 << 30) == VQ_ERR_SHAPE     # pack built for another shape
    pack.data = P + 4
    assert gemv(d, ws=P, ws_bytes=need) == VQ_ERR_ALIGN
    # the packer itself
    out = np.empty(buf.size + 16, dtype=np.uint8)
    hd = vq_weight_t(128, 512, 8, 16, 1, 65536, w.codes.ctypes.data, None, None, None)
    pk = vq_gemv_pack_t()
    assert lib.vq_gemv_prepack(ctypes.byref(hd), None, buf.size, ctypes.byref(pk)) == VQ_ERR_NULL
    aligned = out.ctypes.data + (-out.ctypes.data) % 16
    assert lib.vq_gemv_prepack(ctypes.byref(hd), aligned, buf.size - 1, ctypes.byref(pk)) == VQ_ERR_WORKSPACE
    assert lib.vq_gemv_prepack(ctypes.byref(hd), aligned + 1, buf.size, ctypes.byref(pk)) == VQ_ERR_ALIGN
    hd.v = 4
    assert lib.vq_gemv_prepack(ctypes.byref(hd), aligned, buf.size, ctypes.byref(pk)) == VQ_ERR_UNSUPPORTED
    assert lib.vq_gemv_prepack_bytes(ctypes.byref(hd)) == 0


def test_per_tile_codebook_descriptor_validation():
    assert gemv(weight(K=256, cb_tile_n=32, cb_tile_k=0)) == VQ_ERR_SHAPE    # both or neither
    assert gemv(weight(K=256, cb_tile_n=24, cb_tile_k=64)) == VQ_ERR_SHAPE   # rows per tile: multiple of 16
    assert gemv(weight(K=256, cb_tile_n=32, cb_tile_k=32)) == VQ_ERR_SHAPE   # columns per tile: multiple of 64
    assert gemv(weight(K=320, cb_tile_n=32, cb_tile_k=128)) == VQ_ERR_SHAPE  # K not a whole number of tiles
    assert gemv(weight(K=64 * 600, cb_tile_n=32, cb_tile_k=64)) == VQ_ERR_UNSUPPORTED  # 600 sets of 4 KiB > LDS


def test_packed_12_bit_descriptor_validation():
    ok = dict(code_bits=12, n_entries=4096, n_codebooks=2, K=256)          # 32 positions x 2 = 64 codes per row
    assert gemv(weight(**ok), x=None) == VQ_ERR_NULL                        # descriptor accepted, x missing
    assert gemv(weight(**dict(ok, n_entries=4097))) == VQ_ERR_UNSUPPORTED   # more entries than 12 bits address
    assert gemv(weight(**dict(ok, K=40))) == VQ_ERR_SHAPE                   # 5 x 2 = 10 codes: not whole 12-byte words
    assert gemv(weight(**dict(ok, n_codebooks=4))) == VQ_ERR_UNSUPPORTED    # 256 KiB of codebooks do not fit LDS
    assert gemv(weight(**dict(ok, n_codebooks=3, K=512))) == VQ_ERR_UNSUPPORTED
    assert gemv(weight(**dict(ok, cb_tile_n=32, cb_tile_k=64))) == VQ_ERR_UNSUPPORTED
    assert gemv(weight(code_bits=10)) == VQ_ERR_UNSUPPORTED


def test_gemv_batch_validation():
    lib = vq.lib()
    WP = ctypes.POINTER(vq_weight_t)
    d = weight()
    def batch(ws_list, xs, ys, count=None, ws=None, ws_bytes=0):
        n = len(ws_list)
        wa = (WP * n)(*[ctypes.pointer(w) if w is not None else WP() for w in ws_list])
        xa = (ctypes.c_void_p * n)(*xs)
        ya = (ctypes.c_void_p * n)(*ys)
        return lib.vq_gemv_batch(wa, xa, ya, n if count is None else count, ws, ws_bytes, None)
    assert lib.vq_gemv_batch(None, None, None, 1, None, 0, None) == VQ_ERR_NULL
    assert batch([d], [P], [P], count=0) == VQ_ERR_SHAPE
    assert batch([d] * 5, [P] * 5, [P] * 5) == VQ_ERR_SHAPE             # more than VQ_GEMV_BATCH_MAX
    assert batch([d, None], [P, P], [P, P]) == VQ_ERR_NULL
    assert batch([d, d], [P, None], [P, P]) == VQ_ERR_NULL
    assert batch([d, d], [P, P], [P, P + 2]) == VQ_ERR_ALIGN
    assert batch([d, weight(K=100)], [P, P], [P, P]) == VQ_ERR_SHAPE    # every member is validated
    wa = (WP * 2)(ctypes.pointer(d), ctypes.pointer(d))
    assert lib.vq_gemv_batch_workspace(wa, 2) == 0                      # canonical codes, LDS codebook: no scratch
    assert lib.vq_gemv_batch_workspace(wa, 9) == 0
    assert batch([weight(N=0)], [P], [P]) == 0                          # nothing to do, nothing launched


def test_gemv_sequence_validation():
    """Host-side checks of vq_gemv_sequence: every call and member is validated before anything is launched."""
    import numpy as np
    from paper_2503_02236_amd import workloads as wl
    from paper_2503_02236_amd.binding import vq_gemv_call_t
    lib = vq.lib()
    WP = ctypes.POINTER(vq_weight_t)
    w = wl.make_weight(128, 512, 8, 16, 1, 65536, 0.02, seed=5)
    buf, pack = vq.vq_gemv_prepack(w)
    pack.data = P                                            # a (fake) aligned device address: nothing is launched here
    packed = vq_weight_t(w.N, w.K, 8, 16, 1, 65536, None, P, None, ctypes.pointer(pack))
    canonical = weight()

    def call(ws_list, xs, ys, count=None):
        n = len(ws_list)
        c = vq_gemv_call_t()
        c._keep = ((WP * n)(*[ctypes.pointer(x) if x is not None else WP() for x in ws_list]),
                   (ctypes.c_void_p * n)(*xs), (ctypes.c_void_p * n)(*ys))
        c.w, c.x, c.y = (ctypes.cast(c._keep[0], ctypes.POINTER(WP)), ctypes.cast(c._keep[1], ctypes.POINTER(ctypes.c_void_p)),
                         ctypes.cast(c._keep[2], ctypes.POINTER(ctypes.c_void_p)))
        c.count = n if count is None else count
        return c

    def seq(calls, ws=P, ws_bytes=1 << 30):
        arr = (vq_gemv_call_t * len(calls))(*calls)
        return lib.vq_gemv_sequence(arr, len(calls), ws, ws_bytes, None), lib.vq_gemv_sequence_workspace(arr, len(calls))

    good = call([packed, packed], [P, P], [P, P])
    assert lib.vq_gemv_sequence(None, 1, P, 1 << 30, None) == VQ_ERR_NULL
    arr = (vq_gemv_call_t * 1)(good)
    assert lib.vq_gemv_sequence(arr, 0, P, 1 << 30, None) == VQ_ERR_SHAPE
    need = lib.vq_gemv_sequence_workspace(arr, 1)
    assert need == 2 * (2 * (32 * 128 * 4 + 4096))            # two halves, each the two problems' 32 x 128 partial sums (+ 4 KiB each)
    assert seq([good], ws=None)[0] == VQ_ERR_WORKSPACE
    assert seq([good], ws_bytes=need - 1)[0] == VQ_ERR_WORKSPACE
    assert seq([good], ws=P + 4)[0] == VQ_ERR_ALIGN
    assert seq([good, call([canonical], [P], [P])]) == (VQ_ERR_UNSUPPORTED, 0)     # a member without re-tiled codes
    assert seq([call([packed], [P], [P], count=0)]) == (VQ_ERR_SHAPE, 0)
    assert seq([call([packed] * 5, [P] * 5, [P] * 5)]) == (VQ_ERR_SHAPE, 0)
    assert seq([good, call([packed, None], [P, P], [P, P])]) == (VQ_ERR_NULL, 0)
    assert seq([call([packed], [None], [P])]) == (VQ_ERR_NULL, 0)
    assert seq([call([packed], [P], [P + 2])]) == (VQ_ERR_ALIGN, 0)
    # several streams: the struct is validated before any event or stream is touched
    from paper_2503_02236_amd.binding import vq_side_streams_t
    side = vq_side_streams_t()
    f = lib.vq_gemv_sequence_streams
    assert lib.vq_gemv_sequence_streams_workspace(arr, 1, 1) == need
    assert lib.vq_gemv_sequence_streams_workspace(arr, 1, 0) == 0 and lib.vq_gemv_sequence_streams_workspace(arr, 1, 9) == 0
    two = (vq_gemv_call_t * 2)(good, good)
    assert lib.vq_gemv_sequence_streams_workspace(two, 2, 2) == 2 * need          # one run per stream, two halves each
    assert lib.vq_gemv_sequence_streams_workspace(two, 2, 4) == 2 * need          # runs without calls need nothing
    side.n = 8
    assert f(arr, 1, P, 1 << 30, None, ctypes.byref(side)) == VQ_ERR_SHAPE
    side.n = -1
    assert f(arr, 1, P, 1 << 30, None, ctypes.byref(side)) == VQ_ERR_SHAPE
    side.n = 1
    assert f(arr, 1, P, 1 << 30, None, ctypes.byref(side)) == VQ_ERR_NULL           # no start event
    side.start = P
    assert f(arr, 1, P, 1 << 30, None, ctypes.byref(side)) == VQ_ERR_NULL           # no side stream / done event
    side.n = 0
    assert f(arr, 1, None, 0, None, ctypes.byref(side)) == VQ_ERR_WORKSPACE         # n = 0: the one-stream call


def test_gemv_pipeline_validation():
    """Host-side checks of vq_gemv_pipeline_*: everything is validated before any GPU call; no handle on failure."""
    from paper_2503_02236_amd import workloads as wl
    from paper_2503_02236_amd.binding import vq_gemv_call_t
    lib = vq.lib()
    WP = ctypes.POINTER(vq_weight_t)
    w = wl.make_weight(128, 512, 8, 16, 1, 65536, 0.02, seed=5)
    buf, pack = vq.vq_gemv_prepack(w)
    pack.data = P                                            # a (fake) aligned device address: nothing is launched here
    packed = vq_weight_t(w.N, w.K, 8, 16, 1, 65536, None, P, None, ctypes.pointer(pack))
    canonical = weight()

    def call(ws_list, xs, ys):
        n = len(ws_list)
        c = vq_gemv_call_t()
        c._keep = ((WP * n)(*[ctypes.pointer(x) for x in ws_list]), (ctypes.c_void_p * n)(*xs), (ctypes.c_void_p * n)(*ys))
        c.w, c.x, c.y = (ctypes.cast(c._keep[0], ctypes.POINTER(WP)), ctypes.cast(c._keep[1], ctypes.POINTER(ctypes.c_void_p)),
                         ctypes.cast(c._keep[2], ctypes.POINTER(ctypes.c_void_p)))
        c.count = n
        return c

    def create(calls, ws=P, ws_bytes=1 << 30):                # (P is 256-byte aligned)
        arr = (vq_gemv_call_t * len(calls))(*calls)
        h = ctypes.c_void_p(1)
        st = lib.vq_gemv_pipeline_create(arr, len(calls), ws, ws_bytes, None, ctypes.byref(h))
        assert h.value is None                               # every failure leaves a null handle
        return st, lib.vq_gemv_pipeline_workspace(arr, len(calls))

    assert P % 256 == 0
    good = call([packed, packed], [P, P], [P, P])
    arr = (vq_gemv_call_t * 1)(good)
    need = lib.vq_gemv_pipeline_workspace(arr, 1)
    # status words (256 B), a table of 2 problems (rounded to 256 B), 32 x 1 partial sums for each of 128 rows, twice
    assert need > 256 + 2 * 32 * 128 * 4 and need % 256 == 0
    h = ctypes.c_void_p()
    assert lib.vq_gemv_pipeline_create(arr, 1, P, 1 << 30, None, None) == VQ_ERR_NULL
    assert lib.vq_gemv_pipeline_create(None, 1, P, 1 << 30, None, ctypes.byref(h)) == VQ_ERR_NULL
    assert lib.vq_gemv_pipeline_create(arr, 0, P, 1 << 30, None, ctypes.byref(h)) == VQ_ERR_SHAPE
    assert create([good], ws=None) == (VQ_ERR_WORKSPACE, need)
    assert create([good], ws_bytes=need - 1) == (VQ_ERR_WORKSPACE, need)
    assert create([good], ws=P + 16) == (VQ_ERR_ALIGN, need) # 16-byte aligned is not enough here
    assert create([good, call([canonical], [P], [P])]) == (VQ_ERR_UNSUPPORTED, 0)
    assert create([call([packed], [None], [P])]) == (VQ_ERR_NULL, 0)
    assert create([call([packed], [P], [P + 2])]) == (VQ_ERR_ALIGN, 0)
    assert lib.vq_gemv_pipeline_run(None, None) == VQ_ERR_NULL
    st = ctypes.c_int(7)
    assert lib.vq_gemv_pipeline_status(None, None, ctypes.byref(st)) == VQ_ERR_NULL
    lib.vq_gemv_pipeline_destroy(None)                       # allowed


def test_gemv_pipeline_small_codebook_list_validation():
    """vq_gemv_pipeline_* with canonical uint8 weights of small codebooks (the second kind of list): the workspace is
    the problem table alone; lists that mix kinds or codebook counts are refused before any GPU call."""
    from paper_2503_02236_amd import workloads as wl
    from paper_2503_02236_amd.binding import vq_gemv_call_t
    lib = vq.lib()
    WP = ctypes.POINTER(vq_weight_t)

    def call(ws_list, xs, ys):
        n = len(ws_list)
        c = vq_gemv_call_t()
        c._keep = ((WP * n)(*[ctypes.pointer(x) for x in ws_list]), (ctypes.c_void_p * n)(*xs), (ctypes.c_void_p * n)(*ys))
        c.w, c.x, c.y = (ctypes.cast(c._keep[0], ctypes.POINTER(WP)), ctypes.cast(c._keep[1], ctypes.POINTER(ctypes.c_void_p)),
                         ctypes.cast(c._keep[2], ctypes.POINTER(ctypes.c_void_p)))
        c.count = n
        return c

    def create(calls, ws=P, ws_bytes=1 << 20):
        arr = (vq_gemv_call_t * len(calls))(*calls)
        h = ctypes.c_void_p(1)
        st = lib.vq_gemv_pipeline_create(arr, len(calls), ws, ws_bytes, None, ctypes.byref(h))
        assert h.value is None
        return st, lib.vq_gemv_pipeline_workspace(arr, len(calls))

    two = weight(N=4096, K=4096, n_codebooks=2)
    one = weight(N=300, K=1024, n_codebooks=1, n_entries=64)
    odd_k = weight(N=300, K=1000, n_codebooks=2)              # K not a multiple of 64: not this kind (and not re-tiled)
    wide = weight(N=300, K=16384, n_codebooks=2)              # x does not fit next to the codebook copies
    w16 = wl.make_weight(128, 512, 8, 16, 1, 65536, 0.02, seed=5)
    buf, pack = vq.vq_gemv_prepack(w16)
    pack.data = P
    packed = vq_weight_t(w16.N, w16.K, 8, 16, 1, 65536, None, P, None, ctypes.pointer(pack))
    good = [call([two, two, two], [P, P, P], [P, P, P]), call([two], [P], [P])]
    need = 256                                                # four table entries of 56 bytes, rounded up to 256
    assert create(good, ws=None) == (VQ_ERR_WORKSPACE, need)
    assert create(good, ws_bytes=need - 1) == (VQ_ERR_WORKSPACE, need)
    assert create(good, ws=P + 16) == (VQ_ERR_ALIGN, need)
    assert create([call([two], [P + 2], [P])]) == (VQ_ERR_ALIGN, 0)
    assert create([call([two], [None], [P])]) == (VQ_ERR_NULL, 0)
    assert create([call([two, one], [P, P], [P, P])]) == (VQ_ERR_UNSUPPORTED, 0)     # one and two codebooks in a list
    assert create([call([two], [P], [P]), call([packed], [P], [P])]) == (VQ_ERR_UNSUPPORTED, 0)   # the two kinds mixed
    assert create([call([two, odd_k], [P, P], [P, P])]) == (VQ_ERR_UNSUPPORTED, 0)
    assert create([call([wide], [P], [P])]) == (VQ_ERR_UNSUPPORTED, 0)
    assert create([call([one], [P], [P])], ws=None) == (VQ_ERR_WORKSPACE, 256)       # a single-codebook list is fine


def test_probe_argument_validation():
    lib = vq.lib()
    assert lib.vq_probe_copy(None, P, 16, None) == VQ_ERR_NULL
    assert lib.vq_probe_copy(P, P, 15, None) == VQ_ERR_SHAPE
    assert lib.vq_probe_read(P + 4, 16, P, None) == VQ_ERR_ALIGN
    assert lib.vq_probe_copy(P, P, 0, None) == 0
    assert lib.vq_probe_mfma(1, 1, 0, None, None) == VQ_ERR_NULL
    assert lib.vq_probe_mfma(-1, 1, 0, P, None) == VQ_ERR_SHAPE
    assert lib.vq_probe_mfma(0, 1, 1, P, None) == 0


def test_binding_refuses_host_tensors():
    import torch
    from paper_2503_02236_amd import workloads as wl
    w, x = wl.config1_tiny()
    wd = vq.VQWeightDev(w.N, w.K, w.v, w.code_bits, torch.from_numpy(w.codes), torch.from_numpy(w.codebooks), None)
    with pytest.raises(ValueError):
        vq.vq_gemv(wd, torch.from_numpy(x))


def test_gemv_pipeline_reports_a_failed_host_allocation(tmp_path):
    """The plan of a list is made in host vectors: where one of their allocations fails, the entry points say so instead of
    letting the exception end a C caller's program.  The n-th allocation fails, for every n until a call gets through."""
    shim = tmp_path / "new.cpp"
    shim.write_text("""#include <cstdlib>
#include <new>
extern "C" { long new_fails_in = -1; }
void *operator new(std::size_t n) {
    if (new_fails_in >= 0 && new_fails_in-- == 0) throw std::bad_alloc();
    if (void *p = std::malloc(n ? n : 1)) return p;
    throw std::bad_alloc();
}
""")
    subprocess.run(["g++", "-shared", "-fPIC", "-O1", str(shim), "-o", str(tmp_path / "libnew.so")], check=True)
    code = """
import ctypes, sys
shim = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)      # in front of libvqmi, whose operator new it becomes
fails_in = ctypes.c_long.in_dll(shim, "new_fails_in")
import paper_2503_02236_amd as vq
from paper_2503_02236_amd.binding import vq_gemv_call_t, vq_weight_t
P, n = 0x10000, 64
w = vq_weight_t(1400, 1088, 8, 8, 2, 256, P, P, None, None)
ptr = (ctypes.POINTER(vq_weight_t) * 1)(ctypes.pointer(w))
xy = (ctypes.c_void_p * 1)(P)
calls = (vq_gemv_call_t * n)()
for c in calls:
    c.w, c.x, c.y, c.count = ctypes.cast(ptr, type(c.w)), ctypes.cast(xy, type(c.x)), ctypes.cast(xy, type(c.y)), 1
lib, h = vq.lib(), ctypes.c_void_p()
query = lambda: lib.vq_gemv_pipeline_workspace(calls, n)
create = lambda: lib.vq_gemv_pipeline_create(calls, n, None, 0, None, ctypes.byref(h))
need = query()
assert need > 72 * 256          # (a list for the kernel that deals out segments)
for call, failed, good in ((query, 0, need), (create, -6, -5)):
    for k in range(100000):
        fails_in.value = k
        got = call()
        left, fails_in.value = fails_in.value, -1
        if left >= 0:           # not reached: the call made k allocations and got through
            assert got == good and k > 5, (got, k)
            break
        assert got == failed and not h.value, (got, k)
print("done")
"""
    r = subprocess.run([sys.executable, "-c", code, str(tmp_path / "libnew.so")], cwd=ROOT, capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout.strip() == "done", r.stderr[-2000:]


def internal(name, *args):
    """A bool of the library's own routing functions (C++ names, exported but not part of the ABI)."""
    f = getattr(vq.lib(), name)
    f.restype = ctypes.c_bool
    return f(*args)


@pytest.mark.parametrize("E", [1, 1000, 1001, 16383, 16385])
def test_one_uint16_codebook_of_any_number_of_entries_takes_the_one_pass_product(E):
    """17 .. 256 tokens: an odd number of 8-byte entries cannot be staged in LDS in 16-byte pieces and is looked up in L2."""
    w = weight(N=4096, K=4096, v=4, code_bits=16, n_entries=E)
    assert internal("_ZN2vq21gemm_skinny_supportedEPK11vq_weight_t", ctypes.byref(w))
    # (vq_gemv keeps such a weight where it fits LDS on the row kernel)
    if E % 2 and E < 16384:
        assert not any(internal("_ZN2vq20gemm_skinny_for_gemvEPK11vq_weight_ti", ctypes.byref(w), bs) for bs in range(1, 17))


@pytest.mark.parametrize("kw", [dict(v=8, code_bits=12, n_codebooks=2, n_entries=4096), dict(v=4, code_bits=16, n_entries=65536),
                                dict(v=4, code_bits=8, n_codebooks=2), dict(v=8, code_bits=16, n_codebooks=2, n_entries=2048)])
def test_more_than_256_tokens_without_a_two_stage_product_take_one_pass(kw):
    """K % 64 == 32: the two-stage product does not exist, and 16 tokens a launch would read all codes again and again."""
    one_pass = lambda w, M: internal("_ZN2vq13gemm_one_passEPK11vq_weight_ti", ctypes.byref(w), M)  # noqa: E731
    for M in (17, 256, 257, 2048, 1 << 20):
        assert one_pass(weight(N=4096, K=4128, **kw), M), M
        assert vq.lib().vq_gemm_workspace(ctypes.byref(weight(N=4096, K=4128, **kw)), M) == 0
    assert not one_pass(weight(N=4096, K=4128, **kw), 16)
    # with both ways open a large product keeps the two stages
    assert not one_pass(weight(N=4096, K=4096, **kw), 2048) and one_pass(weight(N=4096, K=4096, **kw), 256)


@pytest.mark.parametrize("kw,n_new,kernel", [
    # prompts of 256 entries, whatever the head size and the groups
    (dict(B=2, H=32, D=128, v=4), 2048, "matrix"), (dict(B=2, H=32, D=96, v=4), 2048, "matrix"), (dict(B=1, H=8, D=80, v=8, cb_groups=2), 300, "matrix"),
    (dict(B=2, H=32, D=192, v=2, cb_groups=32), 100, "matrix"),
    # small codebooks: all entries, a lane per sub-vector
    (dict(B=2, H=32, D=128, v=4, n_entries=16), 2048, "lane"), (dict(B=2, H=32, D=128, v=8, n_entries=8), 2048, "lane"),
    (dict(B=2, H=32, D=128, v=4, n_entries=64), 2048, "matrix"), (dict(B=64, H=32, D=128, v=4, n_entries=16), 5, "lane"),
    # decode steps: a few sequences scan, many do not (their launch is bound by instructions, not by the chain of one item)
    (dict(B=3, H=32, D=128, v=4, cb_groups=32), 1, "scan"), (dict(B=2, H=32, D=128, v=4), 1, "lane"), (dict(B=64, H=32, D=128, v=4), 1, "matrix"),
    (dict(B=64, H=32, D=128, v=4), 5, "matrix"), (dict(B=16, H=32, D=128, v=4, cb_groups=32), 4, "scan"), (dict(B=16, H=32, D=128, v=4, cb_groups=32), 16, "matrix"),
])
def test_kv_quantize_kernel_follows_the_amount_of_work(kw, n_new, kernel):
    f = vq.lib()._ZN2vq21kv_quantize_kernel_ofEPK7vq_kv_ti
    assert f(ctypes.byref(kvdesc(**{**dict(T=4096), **kw})), n_new) == ("scan", "lane", "matrix").index(kernel)


def kv_plan(kw, n_new):
    out = (ctypes.c_int * 5)()
    vq.lib()._ZN2vq19kv_quantize_plan_ofEPK7vq_kv_tiPi(ctypes.byref(kvdesc(**{**dict(T=4096, D=128), **kw})), n_new, out)
    return out


# measured, us: one workgroup per token range / the shared one
@pytest.mark.parametrize("kw,n_new,share", [
    (dict(B=1, H=88, D=64, v=4, cb_groups=4), 1, 1), (dict(B=1, H=74, D=64, v=8), 2, 1), (dict(B=1, H=128, v=8), 1, 1),           # 3.18 / 3.47, 3.37 / 3.66, 3.46 / 3.66
    (dict(B=1, H=28, D=64, v=4), 1, 2), (dict(B=1, H=32, v=4, cb_groups=32), 1, 4), (dict(B=3, H=32, v=4, cb_groups=32), 1, 4),    # 5.0 / 3.0, 5.0 / 4.1 (shared by two 4.3)
    (dict(B=8, H=32, v=4, cb_groups=32), 1, 1),                                                                                   # 6.6 / 6.7
])
def test_kv_quantize_shares_a_token_range_where_that_is_faster(kw, n_new, share):
    out = kv_plan(kw, n_new)
    assert out[0] == 0 and out[4] == share


# measured, us: matrix cores or lanes / the scan that workgroups share
@pytest.mark.parametrize("kw,n_new,kernel", [
    (dict(B=1, H=22, v=4, cb_groups=32), 6, "scan"), (dict(B=1, H=32, v=2, cb_groups=64, n_entries=128), 9, "scan"),   # 13.4 / 5.1, 24.0 / 9.9
    (dict(B=1, H=4, v=4, cb_groups=32), 10, "scan"), (dict(B=1, H=6, v=8), 2, "scan"),                                 # 13.1 / 6.6, 4.3 / 2.7
    (dict(B=8, H=32, v=4, cb_groups=32), 16, "matrix"),                                                                # more workgroups than the chip holds at once
])
def test_kv_quantize_takes_the_fastest_kernel(kw, n_new, kernel):
    f = vq.lib()._ZN2vq21kv_quantize_kernel_ofEPK7vq_kv_ti
    assert f(ctypes.byref(kvdesc(**{**dict(T=4096, D=128), **kw})), n_new) == ("scan", "lane", "matrix").index(kernel)


def test_gemv_takes_the_faster_of_two_kernels_at_the_lines_between_them():
    """Routes on both sides of a line; each was measured as the faster one there."""
    for_gemv = lambda bs, **kw: internal("_ZN2vq20gemm_skinny_for_gemvEPK11vq_weight_ti", ctypes.byref(weight(**kw)), bs)  # noqa: E731
    assert for_gemv(16, N=4096, K=11008, n_codebooks=2) and not for_gemv(13, N=4096, K=11008, n_codebooks=2)
    assert not for_gemv(16, N=11008, K=4096, n_codebooks=2) and not for_gemv(16, N=4096, K=1024)
    assert for_gemv(14, N=1024, K=2048) and not for_gemv(14, N=1024, K=2048, v=4) and for_gemv(14, N=1024, K=4096, v=4)
    assert not for_gemv(14, N=4096, K=4096, v=4, n_codebooks=2) and for_gemv(14, N=3000, K=6400, v=4, n_codebooks=2)


def test_staging_of_large_codebooks_counts_in_the_choice_of_the_product():
    one_pass = lambda M, **kw: internal("_ZN2vq13gemm_one_passEPK11vq_weight_ti", ctypes.byref(weight(**kw)), M)  # noqa: E731
    big = dict(code_bits=12, n_codebooks=2, n_entries=4096)      # 128 KiB of codebooks to stage in every workgroup
    assert one_pass(1024, N=1000, K=512, n_codebooks=2) and not one_pass(1024, N=1000, K=512, **big) and one_pass(257, N=1000, K=512, **big)


# measured, tiles of 48 tokens / the other, us
@pytest.mark.parametrize("kw,M,tile", [
    (dict(N=4096, K=4096, n_codebooks=2), 77, (2, 3)), (dict(N=4096, K=4096, n_codebooks=2), 48, (1, 3)),                # 11.3 / 12.8, 9.2 / 10.4
    (dict(N=4096, K=11008, v=4), 46, (2, 2)), (dict(N=1322, K=11008, v=4), 105, (2, 2)),   # 16.5 / 15.8, 16.3 / 15.4
    (dict(N=4096, K=11008, v=4, n_codebooks=2), 46, (1, 3)),
])
def test_one_pass_product_takes_48_tokens_where_that_is_faster(kw, M, tile):
    f = vq.lib()._ZN2vq19gemm_skinny_tile_ofEPK11vq_weight_ti
    assert divmod(f(ctypes.byref(weight(**kw)), M), 16) == tile


# measured, one pass / two stages, us
@pytest.mark.parametrize("kw,M,one", [
    # more than one round of large tiles: 63.5 / 38.5, 56.5 / 42.0, 63.2 / 42.5 (per-tile codebooks)
    (dict(N=11008, K=2112, n_codebooks=2), 327, False), (dict(N=11008, K=1408), 507, False),
    (dict(N=4096, K=4608, n_codebooks=2, cb_tile_n=256, cb_tile_k=512), 528, False),
    # many lookups of codebooks that no L1 holds, a weight beyond the caches: 149 / 230, 167 / 232; 41.4 / 58.8 with few rows
    (dict(N=11008, K=10560, n_codebooks=2, code_bits=16, n_entries=4096), 317, True), (dict(N=11008, K=11008, n_codebooks=2, code_bits=16, n_entries=4096), 275, True),
    (dict(N=554, K=11008, v=4, n_codebooks=2, code_bits=16, n_entries=1000), 1517, True),
    # the two stages write an odd number of rows element by element: 39.4 / 48.6
    (dict(N=645, K=11008, v=4, n_codebooks=2), 981, True),
])
def test_more_than_256_tokens_take_the_faster_of_the_two_products(kw, M, one):
    assert internal("_ZN2vq13gemm_one_passEPK11vq_weight_ti", ctypes.byref(weight(**kw)), M) == one


@pytest.mark.parametrize("kw,copies", [
    (dict(B=16, H=32, T=4096), True), (dict(B=8, H=32, T=8192), True), (dict(B=33, H=30, T=4096), True),   # whole rounds of long ranges
    (dict(B=3, H=32, T=1500), False),        # 160 workgroups (pairs of batch entries would be 192)
    (dict(B=5, H=32, T=16000), False),       # a round of 256 workgroups and one of 64
    (dict(B=32, H=32, T=64), False), (dict(B=16, H=32, T=3001), False),          # more to stage than to attend
    (dict(B=16, H=32, T=4096, n_entries=64), False), (dict(B=16, H=32, T=4096, cb_groups=32), False), (dict(B=16, H=32, T=4096, v=8), False),
])
def test_attn_copies_of_a_codebook_are_for_long_ranges_in_whole_rounds(kw, copies):
    assert internal("_ZN2vq15attn_replicatedEPK7vq_kv_t", ctypes.byref(kvdesc(**kw))) == copies


def test_dequantization_in_eights_is_for_the_formats_it_is_faster_for():
    eights = lambda **kw: internal("_ZN2vq17dequant_in_eightsEPK11vq_weight_t", ctypes.byref(weight(**{**dict(N=4096, K=4096), **kw})))  # noqa: E731
    assert eights() and eights(code_bits=16, n_entries=65536) and eights(code_bits=12, n_codebooks=2) and eights(code_bits=12, v=4)
    assert not eights(code_bits=12) and not eights(N=300, K=1024) and not eights(n_codebooks=3)


@pytest.mark.parametrize("n,N,K,R,table", [(100, 512, 12288, 2, False), (48, 1024, 11008, 2, False), (48, 4096, 4096, 2, True),
                                           (48, 4096, 4096, 1, True), (48, 16000, 512, 1, True), (3, 1000, 1088, 2, False)])
def test_lists_take_the_table_kernel_where_it_is_ahead(n, N, K, R, table):
    """Measured: few rows of a long K are not faster from a table of products, which is formed anew for every slice of K."""
    from paper_2503_02236_amd.binding import vq_gemv_call_t
    w = weight(N=N, K=K, n_codebooks=R)
    ptr, xy = (ctypes.POINTER(vq_weight_t) * 1)(ctypes.pointer(w)), (ctypes.c_void_p * 1)(P)
    calls = (vq_gemv_call_t * n)()
    for c in calls:
        c.w, c.x, c.y, c.count = ctypes.cast(ptr, type(c.w)), ctypes.cast(xy, type(c.x)), ctypes.cast(xy, type(c.y)), 1
    assert internal("_ZN2vq14gemv_lut_worthEPK14vq_gemv_call_ti", calls, n) == table


def test_binding_finds_the_stream_without_the_undocumented_calls_of_torch(monkeypatch):
    from types import SimpleNamespace as obj
    from paper_2503_02236_amd import binding
    monkeypatch.setattr(binding.torch.cuda, "current_stream", lambda: obj(cuda_stream=77))
    assert binding._stream_getter(obj())() == 77
    assert binding._stream_getter(obj(_cuda_getDevice=lambda: 3))() == 77
    assert binding._stream_getter(obj(_cuda_getDevice=lambda: 3, _cuda_getCurrentRawStream=lambda device: 100 + device))() == 103


def test_native_marshalling_is_used_only_where_it_was_built_for(monkeypatch):
    """Its tensor accessors are inlined from torch's headers: a module for another torch, Python or struct layout is left alone, however
    well it loads."""
    import importlib
    import sysconfig
    import types
    from paper_2503_02236_amd import binding
    l = vq.lib()
    built = importlib.import_module("paper_2503_02236_amd._marshal")
    assert built.built_for == binding.marshal_built_for() and built.__file__.endswith(sysconfig.get_config_var("EXT_SUFFIX"))
    for version in (binding.marshal_built_for(), None, ("torch 0",) + binding.marshal_built_for()[1:], binding.marshal_built_for()[:3] + (0,)):
        calls = []
        fake = types.SimpleNamespace(init=lambda *a: calls.append(a))
        if version:
            fake.built_for = version
        monkeypatch.setattr(binding, "_marshal", None)
        monkeypatch.setitem(sys.modules, "paper_2503_02236_amd._marshal", fake)
        binding._load_marshal(l)
        right = version == binding.marshal_built_for()
        assert len(calls) == right and (binding._marshal is fake) == right


@pytest.mark.skipif(not os.path.exists("/opt/rocm/bin/hipcc"), reason="hipcc not available")
def test_library_is_built_without_the_native_marshalling(tmp_path, monkeypatch, capsys):
    """The C library needs hipcc alone: without a host compiler for the binding's native part it is linked all the same, and a native
    part of an earlier build does not stay beside it."""
    from paper_2503_02236_amd import build

    def compile_one(src, extra):
        obj = str(tmp_path / (src + ".o"))
        subprocess.run([build.HIPCC, "-fPIC", "-x", "c", "-c", "/dev/null", "-o", obj], check=True)
        return obj
    stale = tmp_path / "_marshal.so"
    stale.write_text("stale")
    for name, value in (("SOURCES", ["one.hip"]), ("_compile", compile_one), ("OBJ", str(tmp_path)), ("LIB", str(tmp_path / "lib.so")), ("MARSHAL", str(stale))):
        monkeypatch.setattr(build, name, value)
    monkeypatch.setenv("CXX", "/bin/false")
    assert build.build() == str(tmp_path / "lib.so") and (tmp_path / "lib.so").exists() and not stale.exists()
    assert "marshal.cpp" in capsys.readouterr().err


@pytest.mark.skipif(not os.path.exists("/opt/rocm/bin/hipcc"), reason="hipcc not available")
@pytest.mark.parametrize("how", ["path", "name", "link"])
def test_native_marshalling_finds_the_headers_beside_the_compiler(tmp_path, monkeypatch, how):
    """HIPCC may be a path, a name on PATH, or a link to the compiler: the HIP headers are those beside the compiler itself."""
    from paper_2503_02236_amd import build
    hipcc = "/opt/rocm/bin/hipcc"
    if how == "link":
        os.symlink(hipcc, tmp_path / "hipcc")
        hipcc = str(tmp_path / "hipcc")
    monkeypatch.setattr(build, "HIPCC", "hipcc" if how == "name" else hipcc)
    monkeypatch.setenv("PATH", "/opt/rocm/bin" + os.pathsep + os.environ["PATH"])
    monkeypatch.setattr(build, "MARSHAL", str(tmp_path / "_marshal.so"))
    script = tmp_path / "cxx"
    script.write_text("#!/bin/sh\nfor a in \"$@\"; do case $a in -isystem*) [ -f \"${a#-isystem}/hip/hip_runtime.h\" ] && echo found > \"%s\";; esac; done\nexit 1\n" % (tmp_path / "seen"))
    script.chmod(0o755)
    monkeypatch.setenv("CXX", str(script))
    with pytest.raises(RuntimeError):
        build._build_marshal()
    assert (tmp_path / "seen").exists()
