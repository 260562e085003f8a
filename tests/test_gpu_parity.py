"""GPU parity: every entry point of libvqmi, called through the C ABI, against the CPU oracle
on the same seeded inputs.

Bars: dequantized tiles bit-exact; products and attention within relative L2 <= 2e-3 and
max-abs <= 1e-2 * RMS(oracle output) of the un-rounded fp64 oracle.
"""
import ctypes

import numpy as np
import pytest
import torch

import oracle
import paper_2503_02236_amd as vq
from paper_2503_02236_amd import workloads as wl

pytestmark = pytest.mark.gpu

REL_L2 = 2e-3
MAX_ABS_RMS = 1e-2


def assert_close(got_t, want, what=""):
    got = got_t.float().cpu().numpy().astype(np.float64)
    assert got.shape == want.shape, (got.shape, want.shape)
    assert np.isfinite(got).all(), what
    rel = np.linalg.norm(got - want) / max(np.linalg.norm(want), 1e-300)
    rms = np.sqrt(np.mean(want ** 2))
    mx = np.abs(got - want).max() / max(rms, 1e-300)
    print(f"{what}: rel_l2={rel:.3e} max_abs/rms={mx:.3e}", flush=True)
    assert rel <= REL_L2, (what, rel)
    assert mx <= MAX_ABS_RMS, (what, mx)


def dev_x(x, device):
    return torch.from_numpy(x).to(device)


# ---------------------------------------------------------------- dequantized tiles: bit exact

# weights large enough for the kernel with eight sub-vectors per thread (a ragged last workgroup each): the fp16 tile is the
# fp32 one rounded, bit for bit
@pytest.mark.parametrize("N,K,v,bits,R,E", [(2051, 4160, 8, 16, 1, 65536), (2051, 4160, 8, 8, 2, 256), (1031, 4160, 4, 16, 1, 65536),
                                            (1031, 4160, 4, 8, 2, 256), (2051, 4160, 8, 12, 2, 4096), (1031, 4160, 4, 12, 1, 4096),
                                            (2051, 4160, 8, 16, 2, 3000)])
def test_dequant_large_fp16_is_the_rounded_fp32_tile(gpu_device, N, K, v, bits, R, E):
    wd = vq.weight_to_device(wl.make_weight(N, K, v, bits, R, E, 0.02, seed=60 + v + bits + R), gpu_device)
    half, full = vq.vq_dequant(wd, out_fp32=False), vq.vq_dequant(wd, out_fp32=True)
    assert torch.equal(half.view(torch.int16), full.to(torch.float16).view(torch.int16))


@pytest.mark.parametrize("N,K,v,bits,R,E,sigma", [
    (256, 256, 8, 8, 1, 256, 0.02),        # config 1
    (96, 4096, 8, 16, 1, 65536, 0.02),     # config 2 codebook, a slab of rows
    (80, 4096, 8, 8, 2, 256, 0.01),        # config 3: additive pair
    (64, 1024, 4, 16, 1, 65536, 0.02),     # config 4b
    (33, 72, 4, 8, 3, 100, 0.02),          # ragged everything, three residuals
    (5, 40, 8, 16, 4, 1000, 1e-4),         # mostly subnormal entries
])
def test_dequant_tiles_bit_exact(gpu_device, N, K, v, bits, R, E, sigma):
    w = wl.make_weight(N, K, v, bits, R, E, sigma, seed=7 + N + K)
    wd = vq.weight_to_device(w, gpu_device)
    want32 = oracle.dequant(w.codes, w.codebooks)
    got32 = vq.vq_dequant(wd, out_fp32=True).cpu().numpy()
    assert np.array_equal(got32.view(np.uint32), want32.view(np.uint32))
    got16 = vq.vq_dequant(wd, out_fp32=False).cpu().numpy()
    assert np.array_equal(got16.view(np.uint16), want32.astype(np.float16).view(np.uint16))
    if R == 1:   # one codebook: the tile is the entry's fp16 bits verbatim
        assert np.array_equal(got16.view(np.uint16), w.codebooks[0][w.codes[:, :, 0]].reshape(N, K).view(np.uint16))


@pytest.mark.parametrize("G,v", [(1, 4), (32, 4), (4, 8), (64, 2)])
def test_kv_dequant_bit_exact(gpu_device, G, v):
    kv = wl.make_kv(2, 3, 128, 37, v, 256, G, seed=31 + G)
    kd = vq.kv_to_device(kv, gpu_device)
    for which, codes, cb in ((0, kv.k_codes, kv.k_codebooks), (1, kv.v_codes, kv.v_codebooks)):
        got = vq.vq_kv_dequant(kd, which).cpu().numpy()
        want = oracle.kv_dequant(codes, cb).astype(np.float16)
        assert np.array_equal(got.view(np.uint16), want.view(np.uint16))


# ---------------------------------------------------------------- VQ-gemv

def run_gemv(w, x, device):
    wd = vq.weight_to_device(w, device)
    y = vq.vq_gemv(wd, dev_x(x, device))
    torch.cuda.synchronize()
    return y


def test_gemv_config1_tiny(gpu_device):
    w, x = wl.config1_tiny()
    assert_close(run_gemv(w, x, gpu_device), oracle.gemv(w.codes, w.codebooks, w.scale, x), "C1")


@pytest.mark.parametrize("shape_idx", [0, 1, 2])
def test_gemv_config2_llama7b_full_size(gpu_device, shape_idx):
    w = wl.config2_layer(shape_idx)
    x = wl.make_activations(1, w.K, wl.seed_for(2, shape_idx))
    assert_close(run_gemv(w, x, gpu_device), oracle.gemv(w.codes, w.codebooks, w.scale, x), f"C2[{shape_idx}]")


@pytest.mark.parametrize("shape_idx,bs", [(0, 1), (0, 4), (0, 16), (1, 1), (1, 16), (2, 4), (2, 16)])
def test_gemv_config3_additive_full_size(gpu_device, shape_idx, bs):
    w = wl.config3_layer(shape_idx)
    x = wl.make_activations(bs, w.K, wl.seed_for(3, shape_idx * 100 + bs))
    assert_close(run_gemv(w, x, gpu_device), oracle.gemv(w.codes, w.codebooks, w.scale, x), f"C3[{shape_idx}] bs={bs}")


@pytest.mark.parametrize("N,K,v,bits,R,E,bs,scale", [
    (1, 64, 8, 16, 1, 65536, 1, True),       # a single row
    (19, 4096, 8, 16, 1, 65536, 3, True),    # ragged row count, odd batch
    (130, 11008, 8, 16, 1, 4096, 2, False),  # three K-ranges, last one partly filled
    (77, 8192, 8, 16, 1, 65536, 5, True),    # two K-ranges
    (50, 16384, 8, 16, 1, 65536, 1, True),   # four K-ranges
    (45, 1024, 4, 16, 1, 65536, 7, True),    # v = 4
    (45, 1024, 4, 8, 1, 256, 16, True),      # v = 4, uint8
    (45, 2048, 4, 8, 2, 256, 4, True),       # v = 4 additive
    (45, 2048, 8, 16, 2, 4096, 9, True),     # uint16 additive
    (31, 72, 8, 8, 1, 256, 2, True),         # K not a multiple of the chunk: generic path
    (31, 120, 4, 16, 3, 300, 16, False),     # three residuals: generic path
    (9, 32768, 8, 16, 1, 65536, 1, True),    # very long rows: generic path
])
def test_gemv_shapes_and_edges(gpu_device, N, K, v, bits, R, E, bs, scale):
    sigma = 0.02 / R
    w = wl.make_weight(N, K, v, bits, R, E, sigma, seed=1000 + N + K + bs, with_scale=scale)
    x = wl.make_activations(bs, K, seed=2000 + N + K)
    assert_close(run_gemv(w, x, gpu_device), oracle.gemv(w.codes, w.codebooks, w.scale, x), f"{N}x{K} v{v} R{R} bs{bs}")


# The codebooks on their way to LDS, where the number of 16-byte units is less than, as many as or more than the threads (K = 64: one
# wavefront, 1024: four), and around whole rounds of 4 KiB and pieces of 1 KiB; the last entries are looked up.
@pytest.mark.parametrize("v,R,E", [(8, 1, 1), (8, 1, 63), (8, 1, 64), (8, 1, 65), (8, 1, 255), (8, 1, 256), (8, 1, 257), (8, 1, 1023),
                                   (8, 1, 1024), (8, 1, 1025), (8, 1, 1300), (8, 1, 8192), (8, 2, 511), (4, 1, 514), (4, 2, 2047), (8, 4, 2000)])
@pytest.mark.parametrize("K", [64, 1024])
def test_gemv_codebooks_of_every_length(gpu_device, v, R, E, K):
    w = wl.make_weight(37, K, v, 16, R, E, 0.02, seed=1700 + E + K)
    w.codes[:, -4:, :] = E - 1 - np.arange(4)[:, None] % E
    x = wl.make_activations(2, K, seed=1800 + E)
    assert_close(run_gemv(w, x, gpu_device), oracle.gemv(w.codes, w.codebooks, w.scale, x), f"K {K} v {v} R {R} E {E}")


@pytest.mark.parametrize("v,bits,R,E,sigma", [
    (8, 8, 1, 256, 0.02),       # entries verbatim
    (8, 8, 2, 256, 0.01),       # one fp16 addition = the fp32 sum rounded once
    (8, 8, 4, 256, 0.3),        # four residuals: repeated fp16 additions would differ from the fp32 sum
    (4, 8, 4, 256, 0.3),
    (8, 12, 2, 4096, 0.01),     # packed 12-bit codes
    (8, 12, 4, 2048, 0.3),
])
def test_gemv_matrix_core_operand_is_the_oracle_tile(gpu_device, v, bits, R, E, sigma):
    """The operand the matrix-core gemv consumes, read back through the gemv itself: with one-hot activations
    (token m = unit vector k_m, no scale) y[m][n] = W[n][k_m] exactly, so sixteen columns of the dequantized
    weight come back per call.  They must be the oracle's tile (fp32 sum, r ascending, one rounding to fp16)."""
    N, K = 40, 256
    w = wl.make_weight(N, K, v, bits, R, E, sigma, seed=4700 + R + v + bits, with_scale=False)
    want32 = oracle.dequant(ocodes(w), w.codebooks)
    want = want32.astype(np.float16)
    if R == 4:   # the case must tell the two summations apart: sequential fp16 additions round differently somewhere
        un = (oracle.unpack12(w.codes, N * (K // v) * R).reshape(N, K // v, R) if bits == 12 else w.codes).astype(np.int64)
        seq = w.codebooks[0][un[:, :, 0]].astype(np.float16)
        for r in range(1, R):
            seq = (seq + w.codebooks[r][un[:, :, r]]).astype(np.float16)
        assert (seq.reshape(N, K).view(np.uint16) != want.view(np.uint16)).any()
    wd = vq.weight_to_device(w, gpu_device)
    got = np.empty((N, K), dtype=np.float16)
    for k0 in range(0, K, 16):
        x = np.zeros((16, K), dtype=np.float16)
        x[np.arange(16), k0 + np.arange(16)] = 1.0
        y = vq.vq_gemv(wd, dev_x(x, gpu_device))
        got[:, k0:k0 + 16] = y.cpu().numpy().T
    # (a product with a subnormal fp16 factor may be flushed by the matrix cores: such elements may come back as 0)
    sub = (np.abs(want.astype(np.float32)) < 2.0 ** -14) & (want != 0)
    same = got.view(np.uint16) == want.view(np.uint16)
    print(f"subnormal operands: {int(sub.sum())}, of which returned as zero: {int((sub & ~same).sum())}", flush=True)
    assert same[~sub].all()
    assert (same | (got == 0))[sub].all()


@pytest.mark.parametrize("bs", [1, 5])
def test_gemv_hot_entry_cache_on_reordered_zipf_codes(gpu_device, bs):
    # skewed code usage, entries in arbitrary order, then sorted by use offline: the first entries are
    # served from LDS, the rest from L2; both orders must give the oracle's result
    w = wl.shuffle_entries(wl.make_weight(1000, 2048, 8, 16, 1, 65536, 0.02, seed=9100, zipf_s=1.0), seed=3)
    r = vq.vq_reorder_by_frequency(w)
    x = wl.make_activations(bs, 2048, 9101)
    want = oracle.gemv(w.codes, w.codebooks, w.scale, x)
    assert_close(run_gemv(w, x, gpu_device), want, "zipf shuffled")
    assert_close(run_gemv(r, x, gpu_device), want, "zipf reordered")
    assert 0 < r.hot_entries <= 4096                   # so the reordered weight takes the LDS-cached path
    assert (r.codes < 4096).mean() > 0.6               # and the cache really serves most lookups


def test_gemv_zipf_codes(gpu_device):
    w = wl.config2_layer(0, zipf_s=1.0)
    x = wl.make_activations(1, w.K, 5)
    assert_close(run_gemv(w, x, gpu_device), oracle.gemv(w.codes, w.codebooks, w.scale, x), "C2 zipf")


def test_gemv_is_deterministic_and_leaves_neighbours_alone(gpu_device):
    w = wl.config2_layer(0)
    wd = vq.weight_to_device(w, gpu_device)
    x = dev_x(wl.make_activations(1, w.K, 3), gpu_device)
    buf = torch.full((w.N + 64,), 7.0, dtype=torch.float16, device=gpu_device)
    y = buf[32:32 + w.N].view(1, w.N)
    vq.vq_gemv(wd, x, y=y)
    first = y.clone()
    for _ in range(3):
        vq.vq_gemv(wd, x, y=y)
        assert torch.equal(y, first)
    assert (buf[:32] == 7).all() and (buf[32 + w.N:] == 7).all()


# ---------------------------------------------------------------- VQ-gemv from re-tiled codes

def run_gemv_packed(w, x, device, ws=None):
    wd = vq.weight_to_device(w, device, prepack=True, keep_codes=False)
    assert wd.codes is None                       # the packed path needs no canonical codes
    y = vq.vq_gemv(wd, dev_x(x, device), ws=ws)
    torch.cuda.synchronize()
    return y


@pytest.mark.parametrize("shape_idx", [0, 1, 2])
def test_gemv_packed_config2_full_size(gpu_device, shape_idx):
    w = wl.config2_layer(shape_idx)
    x = wl.make_activations(1, w.K, wl.seed_for(2, shape_idx))
    assert_close(run_gemv_packed(w, x, gpu_device), oracle.gemv(w.codes, w.codebooks, w.scale, x),
                 f"C2 packed[{shape_idx}]")


@pytest.mark.parametrize("N,K,E,scale", [
    (1, 64, 65536, True),         # one row, one sub-vector block
    (63, 1024, 65536, True),      # less than one 64-row group
    (1000, 4096, 65536, False),   # ragged row blocks, no scale
    (300, 2048, 4096, True),      # two slices only
    (257, 16368, 8192, True),     # longest supported rows
    (9000, 512, 65536, True),     # many rows: eighteen groups per workgroup, nine wavefronts with two groups each
    (20000, 128, 65536, True),    # forty groups per workgroup, fourteen wavefronts with up to three groups each
])
def test_gemv_packed_shapes_and_edges(gpu_device, N, K, E, scale):
    w = wl.make_weight(N, K, 8, 16, 1, E, 0.02, seed=3000 + N + K, with_scale=scale)
    x = wl.make_activations(1, K, seed=3100 + N)
    assert_close(run_gemv_packed(w, x, gpu_device), oracle.gemv(w.codes, w.codebooks, w.scale, x),
                 f"packed {N}x{K} E{E}")


def test_gemv_batch_more_groups_than_wavefronts(gpu_device):
    # 20 groups per workgroup: in the batch kernel four wavefronts refill their ring for a second group
    ws = [wl.make_weight(20000, 128, 8, 16, 1, 65536, 0.02, seed=3300 + i) for i in range(2)]
    x = wl.make_activations(1, 128, seed=3310)
    xd = dev_x(x, gpu_device)
    wds = [vq.weight_to_device(w, gpu_device, prepack=True, keep_codes=False) for w in ws]
    ys = vq.vq_gemv_batch(wds, [xd, xd])
    torch.cuda.synchronize()
    for w, wd, y in zip(ws, wds, ys):
        assert_close(y, oracle.gemv(w.codes, w.codebooks, w.scale, x), "batch, 20 groups")
        assert torch.equal(y, vq.vq_gemv(wd, xd))


def test_gemv_skewed_codes_have_no_packed_form_and_run_from_canonical_codes(gpu_device):
    # skewed codes load the codebook slices too unevenly for one common workgroup shape: the re-tiling
    # declines them and vq_gemv serves them from the canonical codes
    w = wl.make_weight(2048, 4096, 8, 16, 1, 65536, 0.02, seed=3000 + 2048 + 4096, zipf_s=1.0)
    assert vq.vq_gemv_prepack(w) == (None, None)
    with pytest.raises(ValueError):
        vq.weight_to_device(w, gpu_device, prepack=True)
    x = wl.make_activations(1, w.K, seed=3100 + 2048)
    y = vq.vq_gemv(vq.weight_to_device(w, gpu_device), dev_x(x, gpu_device))
    torch.cuda.synchronize()
    assert_close(y, oracle.gemv(w.codes, w.codebooks, w.scale, x), "skewed codes, canonical path")


def test_gemv_batch_config2_full_size(gpu_device):
    # the launches bench.py times: query/key/value (3 x 4096x4096) and gate/up (2 x 11008x4096), re-tiled codes
    for shape_idx, count in ((0, 3), (1, 2)):
        ws = [wl.config2_layer(shape_idx, layer=10 + i) for i in range(count)]
        x = wl.make_activations(1, ws[0].K, wl.seed_for(2, 700 + shape_idx))
        xd = dev_x(x, gpu_device)
        wds = [vq.weight_to_device(w, gpu_device, prepack=True, keep_codes=False) for w in ws]
        ys = vq.vq_gemv_batch(wds, [xd] * count)
        torch.cuda.synchronize()
        for i, (w, y) in enumerate(zip(ws, ys)):
            assert_close(y, oracle.gemv(w.codes, w.codebooks, w.scale, x), f"C2 batch[{shape_idx}][{i}]")


def test_gemv_batch_matches_single_calls_and_oracle(gpu_device):
    # query/key/value-like: three matrices, one input; then a mixed batch (different K, one member without a
    # pack, one with an LDS-sized codebook) that takes the one-launch-per-problem route
    x = wl.make_activations(1, 1024, 31)
    xd = dev_x(x, gpu_device)
    ws3 = [wl.make_weight(N, 1024, 8, 16, 1, 65536, 0.02, seed=7300 + i) for i, N in enumerate((768, 768, 300))]
    wds = [vq.weight_to_device(w, gpu_device, prepack=True, keep_codes=False) for w in ws3]
    ys = vq.vq_gemv_batch(wds, [xd, xd, xd])
    again = vq.vq_gemv_batch(wds, [xd, xd, xd])
    torch.cuda.synchronize()
    for w, wd, y, y2 in zip(ws3, wds, ys, again):
        assert_close(y, oracle.gemv(w.codes, w.codebooks, w.scale, x), "batch member")
        assert torch.equal(y, vq.vq_gemv(wd, xd))          # same arithmetic as the single call
        assert torch.equal(y, y2)
    x2 = wl.make_activations(1, 512, 32)
    x2d = dev_x(x2, gpu_device)
    wa = wl.make_weight(200, 512, 8, 16, 1, 65536, 0.02, seed=7310)
    wb = wl.make_weight(130, 512, 8, 8, 2, 256, 0.01, seed=7311)
    mixed = [wds[0], vq.weight_to_device(wa, gpu_device), vq.weight_to_device(wb, gpu_device)]
    ys = vq.vq_gemv_batch(mixed, [xd, x2d, x2d])
    torch.cuda.synchronize()
    for w, xx, y in zip((ws3[0], wa, wb), (x, x2, x2), ys):
        assert_close(y, oracle.gemv(w.codes, w.codebooks, w.scale, xx), "mixed batch member")


@pytest.mark.parametrize("bits,v,R,E,shapes", [
    (8, 8, 2, 256, [(768, 1024), (768, 1024), (300, 1024)]),      # C3-like: two additive 256 x 8 codebooks, ragged last member
    (8, 8, 2, 256, [(2000, 512), (50, 2048)]),                    # different K and very different N in one launch
    (8, 4, 1, 256, [(512, 512), (512, 512), (512, 512), (40, 512)]),
    (12, 8, 2, 4096, [(256, 1024), (512, 1024)]),                 # packed 12-bit codes, 128 KiB of codebooks
    (16, 8, 1, 4096, [(300, 512), (700, 512)]),                   # uint16 codes, a codebook that fits LDS
])
def test_gemv_batch_of_lds_codebook_weights_is_one_launch_with_the_bits_of_single_calls(gpu_device, bits, v, R, E, shapes):
    """vq_gemv_batch on canonical codes whose codebooks live in LDS (the matrix-core gemv): one launch for all
    members; at these sizes K is split over the same number of wavefronts as in a single call, so the bits are
    those of vq_gemv; within tolerance of the oracle."""
    ws = [wl.make_weight(N, K, v, bits, R, E, 0.01, seed=7500 + 10 * bits + i, with_scale=(i % 2 == 0)) for i, (N, K) in enumerate(shapes)]
    xs = [wl.make_activations(1, K, seed=7600 + i) for i, (N, K) in enumerate(shapes)]
    wds = [vq.weight_to_device(w, gpu_device) for w in ws]
    xds = [dev_x(x, gpu_device) for x in xs]
    ys = vq.vq_gemv_batch(wds, xds)
    torch.cuda.synchronize()
    for w, wd, x, xd, y in zip(ws, wds, xs, xds, ys):
        assert torch.equal(y, vq.vq_gemv(wd, xd)), (w.N, w.K)
        codes = oracle.Packed12(w.codes, (w.N, w.K // w.v, w.R)) if bits == 12 else w.codes
        assert_close(y, oracle.gemv(codes, w.codebooks, w.scale, x), f"LDS-codebook batch member {w.N}x{w.K}")


def test_gemv_batch_config3_full_size(gpu_device):
    # the additive configuration at Llama-7B shapes, as bench.py batches it: three 4096 x 4096, two 11008 x 4096
    for shape_idx, count in ((0, 3), (1, 2)):
        ws = [wl.config3_layer(shape_idx, layer=20 + i) for i in range(count)]
        x = wl.make_activations(1, ws[0].K, wl.seed_for(3, 700 + shape_idx))
        xd = dev_x(x, gpu_device)
        wds = [vq.weight_to_device(w, gpu_device) for w in ws]
        ys = vq.vq_gemv_batch(wds, [xd] * count)
        again = vq.vq_gemv_batch(wds, [xd] * count)
        torch.cuda.synchronize()
        for i, (w, wd, y, y2) in enumerate(zip(ws, wds, ys, again)):
            # (the batch may split K over another number of wavefronts than the single call: same products, another
            # order of the fp32 additions; repeated batches are bit-identical)
            assert torch.equal(y, y2)
            assert_close(y, oracle.gemv(w.codes, w.codebooks, w.scale, x), f"C3 batch[{shape_idx}][{i}]")


def test_gemv_sequence_equals_separate_calls(gpu_device):
    """vq_gemv_sequence: the reduction of every launch rides along in the next one.  Mixed shapes (so that the
    pending rows per workgroup go from a few to more than one chunk of 64), single problems and batches, scales
    and none, a launch with fewer workgroups than its predecessor; results bit-identical to vq_gemv_batch."""
    specs = [  # list of calls, each a list of (N, K, E, scale)
        [(4096, 512, 65536, True), (4096, 512, 65536, False), (1000, 512, 65536, True)],
        [(300, 1024, 4096, True)],                      # 10 workgroups only: the 9192 pending rows get the plain reduction kernel
        [(2000, 256, 65536, True), (64, 256, 65536, True)],
        [(11008, 512, 65536, True)],
        [(4096, 1024, 8192, False), (4096, 1024, 65536, True)],
        [(1, 64, 65536, True)],
    ]
    calls, ref = [], []
    seed = 9300
    for spec in specs:
        call = []
        for (N, K, E, sc) in spec:
            seed += 1
            w = wl.make_weight(N, K, 8, 16, 1, E, 0.02, seed=seed, with_scale=sc)
            wd = vq.weight_to_device(w, gpu_device, prepack=True, keep_codes=False)
            x = wl.make_activations(1, K, seed=seed + 500)
            xd = dev_x(x, gpu_device)
            y = torch.full((1, N), 5.0, dtype=torch.float16, device=gpu_device)
            call.append((wd, xd, y))
            ref.append((w, x))
        calls.append(call)
    for rep in range(2):      # twice: the second pass re-uses both halves of the workspace
        vq.vq_gemv_sequence(calls)
        torch.cuda.synchronize()
        flat = [t for c in calls for t in c]
        for (wd, xd, y), (w, x) in zip(flat, ref):
            assert torch.equal(y, vq.vq_gemv(wd, xd)), (w.N, w.K)
            assert_close(y, oracle.gemv(w.codes, w.codebooks, w.scale, x), f"sequence member {w.N}x{w.K}")
            y.fill_(3.0)
    # a sequence of one call is the call itself
    one = [[(calls[0][0][0], calls[0][0][1], torch.empty_like(calls[0][0][2]))]]
    vq.vq_gemv_sequence(one)
    torch.cuda.synchronize()
    assert torch.equal(one[0][0][2], vq.vq_gemv(calls[0][0][0], calls[0][0][1]))


def test_gemv_sequence_llama_block_full_size(gpu_device):
    """One decoder block's projections at full size, as bench.py issues them: (q, k, v), o, (gate, up), down."""
    mats = [wl.config2_layer(i, layer=3) for i in (0, 0, 0, 0, 1, 1, 2)]
    mats = [wl.make_weight(m.N, m.K, 8, 16, 1, 65536, 0.02, seed=9400 + i) for i, m in enumerate(mats)]
    wds = [vq.weight_to_device(m, gpu_device, prepack=True, keep_codes=False) for m in mats]
    xs = {K: dev_x(wl.make_activations(1, K, seed=9450 + K), gpu_device) for K in (4096, 11008)}
    ys = [torch.empty((1, m.N), dtype=torch.float16, device=gpu_device) for m in mats]
    t = [(wd, xs[m.K], y) for wd, m, y in zip(wds, mats, ys)]
    vq.vq_gemv_sequence([t[0:3], t[3:4], t[4:6], t[6:7]])
    torch.cuda.synchronize()
    for (wd, xd, y), m in zip(t, mats):
        assert torch.equal(y, vq.vq_gemv(wd, xd))
        assert_close(y, oracle.gemv(m.codes, m.codebooks, m.scale, xd.cpu().numpy()), f"block member {m.N}x{m.K}")


@pytest.mark.parametrize("n_side", [1, 3])
def test_gemv_sequence_on_several_streams_eager_and_graph(gpu_device, n_side):
    """vq_gemv_sequence_streams: the calls spread over side streams; same bits as separate calls, eagerly and as a
    captured graph replayed several times with eager work and synchronisations in between."""
    calls, flat = [], []
    for c in range(7):                                   # seven calls over 2 or 4 streams: runs of 4 + 3 or 2 + 2 + 2 + 1
        call = []
        for k in range(1 + c % 3):
            N, K = [(4096, 512), (1000, 1024), (2500, 256)][(c + k) % 3]
            w = wl.make_weight(N, K, 8, 16, 1, 65536, 0.02, seed=9600 + 10 * c + k)
            wd = vq.weight_to_device(w, gpu_device, prepack=True, keep_codes=False)
            xd = dev_x(wl.make_activations(1, K, seed=9700 + 10 * c + k), gpu_device)
            call.append((wd, xd, torch.full((1, N), 7.0, dtype=torch.float16, device=gpu_device)))
        calls.append(call)
        flat += call
    want = [vq.vq_gemv(wd, xd).clone() for (wd, xd, _) in flat]
    torch.cuda.synchronize()
    seq = vq.GemvSequence(calls)
    side = vq.SideStreams(n_side, gpu_device)
    ws = vq.new_workspace(seq.workspace_streams(n_side + 1), gpu_device)

    def run():
        st = seq.run_streams(ws.data_ptr(), ws.numel(), side)
        assert st == 0, vq.status_str(st)

    def check(tag):
        torch.cuda.synchronize()
        for (wd, xd, y), w_ in zip(flat, want):
            assert torch.equal(y, w_), tag
            y.fill_(7.0)
        torch.cuda.synchronize()

    run()
    check("eager")
    run()
    check("eager, second time")
    g = torch.cuda.CUDAGraph()
    cap = torch.cuda.Stream()
    with torch.cuda.stream(cap):
        with torch.cuda.graph(g, stream=cap):
            run()
    for rep in range(4):
        g.replay()
        check(f"replay {rep}")
        vq.vq_gemv(flat[0][0], flat[0][1])               # eager work of the program between the replays
        torch.cuda.synchronize()


def _pipeline_case(gpu_device, specs, seed0, reps=2):
    calls, ref = [], []
    seed = seed0
    for spec in specs:
        call = []
        for (N, K, E, sc) in spec:
            seed += 1
            w = wl.make_weight(N, K, 8, 16, 1, E, 0.02, seed=seed, with_scale=sc)
            wd = vq.weight_to_device(w, gpu_device, prepack=True, keep_codes=False)
            x = wl.make_activations(1, K, seed=seed + 500)
            call.append((wd, dev_x(x, gpu_device), torch.full((1, N), 5.0, dtype=torch.float16, device=gpu_device)))
            ref.append((w, x))
        calls.append(call)
    flat = [t for c in calls for t in c]
    want = [vq.vq_gemv(wd, xd).clone() for (wd, xd, _) in flat]
    torch.cuda.synchronize()
    pipe = vq.GemvPipeline(calls)
    for rep in range(reps):                                  # again: the second run re-uses table, workspace and LDS protocol
        assert pipe.run() == 0
        torch.cuda.synchronize()
        assert pipe.status() == 0                            # no wavefront gave up a wait
        for (wd, xd, y), w_, (w, x) in zip(flat, want, ref):
            assert torch.equal(y, w_), (w.N, w.K, rep)       # the additions of vq_gemv in the order of vq_gemv
            if rep == 0:
                assert_close(y, oracle.gemv(w.codes, w.codebooks, w.scale, x), f"pipeline member {w.N}x{w.K}")
            y.fill_(3.0)
    pipe.close()


def _small_codebook_list(gpu_device, R, specs, seed0, subsets):
    calls, ref = [], []
    for i, (N, K, E, sc) in enumerate(specs):
        w = wl.make_weight(N, K, 8, 8, R, E, 0.01, seed=seed0 + i, with_scale=sc)
        x = wl.make_activations(1, K, seed=seed0 + 500 + i)
        calls.append([(vq.weight_to_device(w, gpu_device), dev_x(x, gpu_device),
                       torch.full((1, N), 5.0, dtype=torch.float16, device=gpu_device))])
        ref.append((w, x))
    first = {}
    for sub in subsets:
        pipe = vq.GemvPipeline([calls[i] for i in sub])
        for rep in range(2):                                     # the second run re-uses the table and the LDS contents
            assert pipe.run() == 0
            torch.cuda.synchronize()
            assert pipe.status() == 0
            for i in sub:
                w, x = ref[i]
                y = calls[i][0][2]
                assert_close(y, oracle.gemv(w.codes, w.codebooks, w.scale, x), f"list member {w.N}x{w.K} R={R} of {len(sub)}")
                # the bits do not depend on the run, nor on what else is in the list (every order is fixed per problem)
                assert torch.equal(y, first.setdefault(i, y.clone())), (w.N, w.K, rep, len(sub))
                y.fill_(3.0)
        pipe.close()


def test_gemv_pipeline_small_codebook_lists(gpu_device):
    """vq_gemv_pipeline with canonical uint8 weights of small codebooks: 16 LDS copies of every entry, a list of
    problems in one launch.  Rows that end inside a chunk of 512 positions (K = 1024 + 64, 11008, 2112), three chunks
    (K = 11008, 12288), one row, fewer rows than workgroups, codebooks of 16 / 64 / 128 entries, no scale; lists of 1,
    3, 4 and all problems (1, 2, 4 and 8 groups of workgroups); one and two additive codebooks."""
    _small_codebook_list(gpu_device, 2, [(4096, 4096, 256, True), (300, 1024, 256, False), (11008, 4096, 256, True),
                                         (4096, 11008, 256, True), (1, 512, 256, True), (777, 2112, 64, True),
                                         (513, 12288, 256, True), (2000, 576, 256, True), (64, 8192, 16, False)],
                         9900, [range(9), [0], [0, 1, 2], [6, 4, 3, 8]])
    _small_codebook_list(gpu_device, 1, [(4096, 4096, 256, True), (333, 1088, 256, True), (1000, 11008, 128, False)],
                         9950, [range(3), [2]])


def test_gemv_pipeline_small_codebook_list_of_forty(gpu_device):
    """Forty problems in one list: 32 groups of 8 workgroups (the launch shape of the decoder stack in bench.py), some
    groups with two problems and some with one; shapes cycle through ragged and whole chunks."""
    shapes = [(700, 1088), (512, 512), (1000, 2112), (96, 4096), (2049, 576)]
    specs = [shapes[i % len(shapes)] + (256, i % 3 != 0) for i in range(40)]
    _small_codebook_list(gpu_device, 2, specs, 9600, [range(40), range(33)])


@pytest.mark.parametrize("R,count,shapes", [
    (2, 192, [(1400, 1088), (1024, 2112), (512, 512), (129, 576), (1, 512), (1300, 1408), (8, 1024)]),
    (1, 192, [(1400, 1088), (1024, 2112), (512, 512), (129, 576), (1, 512), (1300, 1408), (8, 1024)]),
    (2, 48, [(2100, 12288), (2100, 11008), (700, 4096)]),         # rows of 2752 bytes: even and odd rows dealt apart
    (2, 48, [(8300, 1088), (1100, 1088)]),                        # rows of 272 bytes: every eighth row
    (1, 48, [(4200, 1280), (16500, 576), (300, 12288)]),          # every fourth (160 bytes), every sixteenth (72)
])
def test_gemv_pipeline_long_small_codebook_lists(gpu_device, R, count, shapes):
    """Lists long enough for the kernel that looks products up in a table: rows that end inside a slice of 64 (or 128)
    positions, fewer rows than a step's 128, one row, rows and codes that start inside a 128-byte line, small codebooks, no
    scale; the same bits on a second run, and entries that no code uses may hold anything."""
    calls, ref = [], []
    for i in range(count):
        N, K = shapes[i % len(shapes)]
        E = (256, 250, 16)[i % 3]
        w = wl.make_weight(N, K, 8, 8, R, E, 0.01, seed=12000 + 100 * R + i, with_scale=(i % 4 != 0))
        if E == 256 and N > 1:
            w.codes[...] = w.codes % 255
            w.codebooks[:, 255, :] = np.float16("nan")
        x = wl.make_activations(1, w.K, seed=12500 + i)
        wd = vq.weight_to_device(w, gpu_device)
        if i % 5 == 1:      # codes that do not start at a line
            flat = torch.zeros(wd.codes.numel() + 16, dtype=torch.uint8, device=gpu_device)
            flat[16:] = wd.codes.reshape(-1)
            wd.codes = flat[16:].view(wd.codes.shape)
        calls.append([(wd, dev_x(x, gpu_device), torch.full((1, N), 5.0, dtype=torch.float16, device=gpu_device))])
        ref.append((w, x))
    pipe = vq.GemvPipeline(calls)
    # (the table of the kernel for short lists is smaller than this)
    assert vq.lib().vq_gemv_pipeline_workspace(pipe.seq.arr, pipe.seq.n) > 72 * 256
    first = []
    for rep in range(2):
        assert pipe.run() == 0
        torch.cuda.synchronize()
        for i, (c, (w, x)) in enumerate(zip(calls, ref)):
            y = c[0][2]
            if rep == 0:
                assert_close(y, oracle.gemv(w.codes, w.codebooks, w.scale, x), f"long list member {i}: {w.N}x{w.K} R={R}")
                first.append(y.clone())
            else:
                assert torch.equal(y, first[i]), i
            y.fill_(3.0)
    pipe.close()


@pytest.mark.parametrize("R", [1, 2])
def test_gemv_pipeline_long_list_infinite_entry_at_the_start_of_a_row(gpu_device, R):
    """A lane whose 16 code bytes lie partly outside its row looks up the row's first codes in place of the missing ones.
    Where the first code names an infinite entry, the row is +-inf, and no zero of the padding may turn that into a NaN:
    rows of 72 (144) bytes, whose ends lie 8 (0) bytes into a chunk of 16, dealt as one run of rows and as every
    sixteenth (eighth)."""
    calls, ref = [], []
    for i in range(48):
        N = (16500, 700)[i % 2]
        w = wl.make_weight(N, 576, 8, 8, R, 256, 0.01, seed=12700 + i, with_scale=(i % 4 != 0))
        w.codes[w.codes == 7] = 8
        w.codes[3::5, 0, R - 1] = 7
        w.codebooks[R - 1, 7, 2] = np.float16(np.inf)
        x = wl.make_activations(1, w.K, seed=12800 + i)
        wd = vq.weight_to_device(w, gpu_device)
        calls.append([(wd, dev_x(x, gpu_device), torch.zeros((1, N), dtype=torch.float16, device=gpu_device))])
        ref.append((w, x))
    pipe = vq.GemvPipeline(calls)
    assert vq.lib().vq_gemv_pipeline_workspace(pipe.seq.arr, pipe.seq.n) > 72 * 256     # (a long list)
    assert pipe.run() == 0
    torch.cuda.synchronize()
    for i, (c, (w, x)) in enumerate(zip(calls, ref)):
        got = c[0][2].float().cpu().numpy()[0]
        want = oracle.gemv(w.codes, w.codebooks, w.scale, x)[0]
        inf = np.arange(w.N) % 5 == 3
        assert np.array_equal(np.isinf(want), inf) and np.array_equal(got[inf], want[inf].astype(np.float32)), i
        assert_close(torch.from_numpy(got[~inf]), want[~inf], f"finite rows of member {i}, R={R}")
    pipe.close()


def test_gemv_pipeline_small_codebook_nan_entries_unused(gpu_device):
    """Entries that no code uses are never multiplied into a result: with NaN in them the outputs stay finite and
    equal those with zeros there (a lane past the end of a ragged row computes with codes that are not its own;
    that value is dropped, not multiplied by zero)."""
    N, K, E = 600, 1088, 256
    w = wl.make_weight(N, K, 8, 8, 2, E, 0.01, seed=9970, with_scale=True)
    w.codes[...] = w.codes % 200                             # entries 200..255 of both codebooks are never used
    x = wl.make_activations(1, K, seed=9971)
    outs = []
    for fill in (0.0, float("nan")):
        w.codebooks[:, 200:, :] = np.float16(fill)
        wd = vq.weight_to_device(w, gpu_device)
        y = torch.full((1, N), 5.0, dtype=torch.float16, device=gpu_device)
        pipe = vq.GemvPipeline([[(wd, dev_x(x, gpu_device), y)]])
        assert pipe.run() == 0
        torch.cuda.synchronize()
        outs.append(y.clone())
        pipe.close()
    assert torch.isfinite(outs[1]).all()
    assert torch.equal(outs[0], outs[1])
    w.codebooks[:, 200:, :] = np.float16(0.0)
    assert_close(outs[0], oracle.gemv(w.codes, w.codebooks, w.scale, x), "nan-entries case")


def test_gemv_pipeline_config3_stack_full_size(gpu_device):
    """Two decoder blocks of the additive 2 x 256 x 8 configuration at full size (4 + 2 + 1 matrices each) as one
    list: sampled rows against the oracle, all rows finite, repeatable."""
    calls, ref = [], []
    for blk in range(2):
        for si, cnt in ((0, 4), (1, 2), (2, 1)):
            N, K = wl.LLAMA7B_SHAPES[si]
            for j in range(cnt):
                w = wl.config3_layer(si, blk * 4 + j)
                x = wl.make_activations(1, K, seed=9990 + len(calls))
                calls.append([(vq.weight_to_device(w, gpu_device), dev_x(x, gpu_device),
                               torch.full((1, N), 5.0, dtype=torch.float16, device=gpu_device))])
                ref.append((w, x))
    pipe = vq.GemvPipeline(calls)
    assert pipe.run() == 0
    torch.cuda.synchronize()
    first = [c[0][2].clone() for c in calls]
    assert pipe.run() == 0
    torch.cuda.synchronize()
    rng = np.random.default_rng(77)
    for c, f, (w, x) in zip(calls, first, ref):
        assert torch.equal(c[0][2], f)
        assert torch.isfinite(f).all()
        rows = np.unique(np.concatenate([rng.integers(0, w.N, 48), [0, w.N - 1]]))
        want = oracle.gemv(w.codes, w.codebooks, w.scale, x, rows=rows)
        assert_close(f[:, torch.from_numpy(rows).to(f.device)], want, f"stack member {w.N}x{w.K}")
    pipe.close()


def test_gemv_pipeline_mixed_shapes(gpu_device):
    """vq_gemv_pipeline: one persistent launch for all products.  One, two and many problems; problems with fewer
    blocks than the launch has workgroups, with one row, without scale, with smaller codebooks (fewer slices), with
    groups longer than one piece (K = 2048: about 11 steps in the longest group); bit-identical to vq_gemv."""
    _pipeline_case(gpu_device, [[(512, 512, 65536, True)]], 9800)
    _pipeline_case(gpu_device, [[(4096, 512, 65536, True)], [(1000, 1024, 65536, False)]], 9810)
    _pipeline_case(gpu_device, [
        [(4096, 512, 65536, True), (4096, 512, 65536, False), (1000, 512, 65536, True)],
        [(300, 1024, 4096, True)],
        [(2000, 256, 65536, True), (64, 256, 65536, True)],
        [(11008, 512, 65536, True)],
        [(4096, 1024, 8192, False), (4096, 2048, 65536, True)],
        [(1, 64, 65536, True)]], 9820)


def test_gemv_pipeline_as_replayed_graph(gpu_device):
    """vq_gemv_pipeline_run captured into a HIP graph (as bench.py times it) and replayed several times with eager
    work and synchronisations in between: every replay gives the bits of vq_gemv."""
    calls, flat = [], []
    for c in range(5):
        call = []
        for k in range(1 + c % 2):
            N, K = [(4096, 512), (1000, 1024), (2500, 256)][(c + k) % 3]
            w = wl.make_weight(N, K, 8, 16, 1, 65536, 0.02, seed=9900 + 10 * c + k)
            wd = vq.weight_to_device(w, gpu_device, prepack=True, keep_codes=False)
            xd = dev_x(wl.make_activations(1, K, seed=9950 + 10 * c + k), gpu_device)
            call.append((wd, xd, torch.full((1, N), 7.0, dtype=torch.float16, device=gpu_device)))
        calls.append(call)
        flat += call
    want = [vq.vq_gemv(wd, xd).clone() for (wd, xd, _) in flat]
    torch.cuda.synchronize()
    pipe = vq.GemvPipeline(calls)

    def check(tag):
        torch.cuda.synchronize()
        assert pipe.status() == 0, tag
        for (wd, xd, y), w_ in zip(flat, want):
            assert torch.equal(y, w_), tag
            y.fill_(7.0)
        torch.cuda.synchronize()

    assert pipe.run() == 0
    check("eager")
    g = torch.cuda.CUDAGraph()
    cap = torch.cuda.Stream()
    with torch.cuda.stream(cap):
        with torch.cuda.graph(g, stream=cap):
            assert pipe.run() == 0
    for rep in range(4):
        g.replay()
        check(f"replay {rep}")
        vq.vq_gemv(flat[0][0], flat[0][1])               # eager work of the program between the replays
        torch.cuda.synchronize()
    del g
    pipe.close()


def test_gemv_pipeline_llama_blocks_full_size(gpu_device):
    """Two decoder blocks at full size, as bench.py issues them (four problem lanes, four row blocks per LDS image,
    K = 11008 in two parts): bit-identical to vq_gemv, within tolerance of the oracle."""
    block = [[(4096, 4096, 65536, True)] * 3, [(4096, 4096, 65536, True)], [(11008, 4096, 65536, True)] * 2,
             [(4096, 11008, 65536, True)]]
    _pipeline_case(gpu_device, block + block, 9850)


def test_gemv_packed_padding_never_touches_a_codebook_entry(gpu_device):
    # entries that no code uses are set to infinity and NaN: padding atoms multiply a zero unit of x with an
    # entry that some code really uses, never with one of these, so every output stays what the oracle says (finite)
    w = wl.make_weight(200, 1024, 8, 16, 1, 65536, 0.02, seed=7400)
    used = np.zeros(65536, dtype=bool)
    used[w.codes.reshape(-1)] = True
    unused = np.flatnonzero(~used)
    assert unused.size > 30000
    w.codebooks[0, unused[0::2]] = np.float16(np.inf)
    w.codebooks[0, unused[1::2]] = np.float16(np.nan)
    if not used[0]:
        assert not np.isfinite(w.codebooks[0, 0]).any()          # entry 0 of slice 0 among them
    x = wl.make_activations(1, w.K, 7401)
    want = oracle.gemv(w.codes, w.codebooks, w.scale, x)
    assert np.isfinite(want).all()
    got = run_gemv_packed(w, x, gpu_device)
    assert torch.isfinite(got).all()
    assert_close(got, want, "packed gemv with non-finite unused entries")


def test_gemv_packed_shared_workspace_determinism_and_canonical_agreement(gpu_device):
    # three layers of different shapes share one workspace, called back to back, twice
    ws_bytes, layers = 0, []
    for si in (0, 1, 2):
        w = wl.config2_layer(si, layer=5)
        wd = vq.weight_to_device(w, gpu_device, prepack=True)
        x = dev_x(wl.make_activations(1, w.K, 40 + si), gpu_device)
        layers.append((w, wd, x))
        ws_bytes = max(ws_bytes, vq.vq_gemv_workspace(wd, 1))
    assert ws_bytes == 32 * 11008 * 4 + 4096   # S x N fp32 partial sums (N a multiple of 64 here), 32 slices of 2048 entries
    ws = vq.new_workspace(ws_bytes, gpu_device)
    outs = [[vq.vq_gemv(wd, x, ws=ws).clone() for (_, wd, x) in layers] for _ in range(3)]
    torch.cuda.synchronize()
    for rep in outs[1:]:
        for a, b in zip(outs[0], rep):
            assert torch.equal(a, b)
    for (w, wd, x), y in zip(layers, outs[0]):
        assert_close(y, oracle.gemv(w.codes, w.codebooks, w.scale, x.cpu().numpy()), "packed shared ws")
        # bs > 1 on the same descriptor takes the canonical-layout path and agrees
        x2 = torch.cat([x, x], dim=0).contiguous()
        y2 = vq.vq_gemv(wd, x2, ws=ws)
        assert (y2[0].float() - y[0].float()).abs().max() <= 2e-2 * y.float().abs().max()
        assert torch.equal(y2[0], y2[1])


# ---------------------------------------------------------------- VQ-gemm

@pytest.mark.parametrize("M,N,K,v,scale", [
    (96, 256, 512, 8, False),
    (300, 200, 1024, 8, True),     # ragged M and N tiles
    (257, 520, 256, 4, True),      # v = 4, ragged
    (32, 64, 64, 8, False),        # one K block
    (7, 40, 128, 8, True),         # small M: row-kernel path
])
def test_gemm_small_full_compare(gpu_device, M, N, K, v, scale):
    w = wl.make_weight(N, K, v, 16, 1, 65536, 0.02, seed=4000 + M + N, with_scale=scale)
    X = wl.make_activations(M, K, seed=4100 + M)
    Y = vq.vq_gemm(vq.weight_to_device(w, gpu_device), dev_x(X, gpu_device))
    torch.cuda.synchronize()
    assert_close(Y, oracle.gemm(w.codes, w.codebooks, w.scale, X), f"gemm {M}x{N}x{K} v{v}")


def test_gemm_other_formats_use_row_path(gpu_device):
    w = wl.make_weight(70, 256, 8, 8, 2, 256, 0.01, seed=4500)
    X = wl.make_activations(40, 256, seed=4501)
    Y = vq.vq_gemm(vq.weight_to_device(w, gpu_device), dev_x(X, gpu_device))
    assert_close(Y, oracle.gemm(w.codes, w.codebooks, w.scale, X), "gemm uint8 R=2")


@pytest.mark.parametrize("M,N,K,v,bits,R,E", [
    (300, 130, 256, 8, 8, 2, 256),      # additive uint8 pairs, ragged tiles
    (513, 257, 192, 4, 16, 3, 500),     # three residual codebooks, v = 4
    (1025, 64, 64, 8, 8, 1, 256),       # one K block, five M tiles
    (700, 200, 320, 8, 8, 1, 256),      # rows of Y 16-byte aligned (vector stores), ragged in M and N
    (257, 136, 128, 4, 8, 2, 64),       # same store path, second N tile holds one 8-column segment
])
def test_gemm_large_m_any_format_two_stage(gpu_device, M, N, K, v, bits, R, E):
    w = wl.make_weight(N, K, v, bits, R, E, 0.02 / R, seed=4700 + M)
    X = wl.make_activations(M, K, seed=4701 + M)
    wd = vq.weight_to_device(w, gpu_device)
    assert vq.vq_gemm_workspace(wd, M) == N * K * 2
    Y = vq.vq_gemm(wd, dev_x(X, gpu_device))
    torch.cuda.synchronize()
    assert_close(Y, oracle.gemm(w.codes, w.codebooks, w.scale, X), f"gemm two-stage {M}x{N}x{K} R{R}")


@pytest.mark.parametrize("N,v", [(4096, 8), (11008, 8), (4096, 4), (11008, 4)])
def test_gemm_config4_full_size_sampled_columns(gpu_device, N, v):
    w = wl.config4_layer(N, v)
    X = wl.make_activations(2048, 4096, wl.seed_for(4, N + v))
    Y = vq.vq_gemm(vq.weight_to_device(w, gpu_device), dev_x(X, gpu_device))
    torch.cuda.synchronize()
    r = np.random.Generator(np.random.PCG64(N + v))
    # stratified: one output column out of every 64 (so every 64-, 128- and 256-column tile of the kernel's
    # tile map holds compared elements), all 2048 tokens of each, plus the edges of the first and last tiles
    n64 = (N + 63) // 64
    strat = np.arange(n64) * 64 + r.integers(0, 64, size=n64)
    rows = np.unique(np.concatenate([strat[strat < N], [0, 31, 32, 255, 256, N - 1, N - 33]]))
    assert len(np.unique(rows // 128)) == (N + 127) // 128
    want = oracle.gemm(w.codes, w.codebooks, w.scale, X, rows=rows)      # all 2048 tokens x sampled columns
    assert_close(Y[:, torch.from_numpy(rows).to(gpu_device)], want, f"C4 N={N} v={v}")
    assert torch.isfinite(Y.float()).all()


# The two-stage product at ragged sizes: three and four codebooks always take it, at any size (one K block, N of one and
# of two tiles, rows of Y 16-byte aligned and not, several M tiles; the tile is chosen by estimated time, test_gemm_tiles runs every one).
@pytest.mark.parametrize("M,N,K,v,bits,R", [(300, 130, 256, 8, 8, 4), (1025, 64, 64, 8, 8, 4), (700, 200, 320, 8, 8, 3), (257, 136, 128, 4, 8, 4),
                                            (257, 520, 256, 4, 16, 3), (1990, 3013, 64, 8, 8, 3), (1990, 3016, 192, 8, 8, 4)])
def test_gemm_two_stage_ragged(gpu_device, M, N, K, v, bits, R):
    w = wl.make_weight(N, K, v, bits, R, 200, 0.02 / R, seed=4760 + M)
    X = wl.make_activations(M, K, seed=4761 + M)
    Y = vq.vq_gemm(vq.weight_to_device(w, gpu_device), dev_x(X, gpu_device))
    assert_close(Y, oracle.gemm(w.codes, w.codebooks, w.scale, X), f"gemm two-stage {M}x{N}x{K} R{R}")


# The two stages by themselves: the weight in operand order (16-column strips, the last one narrower) holds the bits of vq_dequant,
# every code format, with eight units of 8 k per thread (large) and with two (small)
@pytest.mark.parametrize("N,K", [(1, 64), (37, 192), (130, 320), (2051, 4160), (2056, 4096)])
@pytest.mark.parametrize("v,bits,R,E", [(8, 8, 1, 256), (8, 8, 2, 200), (4, 8, 2, 256), (4, 8, 4, 64), (8, 16, 1, 65536), (4, 16, 1, 5001), (4, 16, 3, 500),
                                        (8, 12, 1, 4096), (8, 12, 2, 4096), (4, 12, 2, 2000), (8, 8, 3, 256)])
def test_dequant_in_operand_order(gpu_device, N, K, v, bits, R, E):
    w = vq.weight_to_device(wl.make_weight(N, K, v, bits, R, E, 0.05, seed=4780 + N), gpu_device)
    rows = vq.vq_dequant(w, out_fp32=False).cpu().numpy()
    got = torch.full((N * K + 64,), 7.0, dtype=torch.float16, device=gpu_device)
    f = vq.lib()._ZN2vq22launch_dequant_orderedEPK11vq_weight_tPDF16_P12ihipStream_t
    assert f(ctypes.byref(w.desc()), ctypes.c_void_p(got.data_ptr()), ctypes.c_void_p(0)) == 0
    torch.cuda.synchronize()
    n, k = np.arange(N)[:, None], np.arange(K)[None, :]
    c = np.minimum(16, N - n // 16 * 16)
    at = 16 * K * (n // 16) + 32 * c * (k // 32) + 8 * c * (k % 32 // 8) + 8 * (n % 16) + k % 8
    got = got.cpu().numpy()
    assert len(np.unique(at)) == N * K and np.array_equal(got[at].view(np.uint16), rows.view(np.uint16)) and (got[N * K:] == 7).all()


# ... and every tile of the product, at the edges of tiles, strips, fragments and the ring of stages
@pytest.mark.parametrize("M,N,K", [(1, 1, 64), (70, 37, 128), (129, 264, 192), (257, 72, 320), (300, 513, 448), (513, 200, 1024)])
@pytest.mark.parametrize("pick", range(8))
def test_gemm_tiles(gpu_device, M, N, K, pick):
    g = torch.Generator(device=gpu_device).manual_seed(4790 + M + pick)
    X = torch.randn((M, K), generator=g, device=gpu_device).to(torch.float16)
    W = (torch.randn((N, K), generator=g, device=gpu_device) * 0.05).to(torch.float16)
    scale = (torch.rand(N, generator=g, device=gpu_device) + 0.5).to(torch.float16) if pick % 2 or M == 513 else None
    n, k = torch.arange(N, device=gpu_device)[:, None], torch.arange(K, device=gpu_device)[None, :]
    c = torch.clamp(N - n // 16 * 16, max=16)
    ordered = torch.empty(N * K, dtype=torch.float16, device=gpu_device)
    ordered[16 * K * (n // 16) + 32 * c * (k // 32) + 8 * c * (k % 32 // 8) + 8 * (n % 16) + k % 8] = W
    Y = torch.full((M + 1, N), 7.0, dtype=torch.float16, device=gpu_device)
    ptr = lambda t: ctypes.c_void_p(0 if t is None else t.data_ptr())  # noqa: E731
    torch.cuda.synchronize()
    assert vq.lib()._ZN2vq17launch_gemm_tilesEPKDF16_S1_S1_PDF16_iiiiP12ihipStream_t(ptr(X), ptr(ordered), ptr(scale), ptr(Y), M, N, K, pick, ptr(None)) == 0
    torch.cuda.synchronize()
    want = X.double().cpu().numpy() @ W.double().cpu().numpy().T * (1 if scale is None else scale.double().cpu().numpy())
    assert_close(Y[:M], want, f"tile {pick} {M}x{N}x{K}")
    assert (Y[M] == 7).all()


# The second stage for a K beyond 2^22 by itself, at the edges of its two tiles (128 x 128, and 256 x 128 where the last sizes fill the chip
# with them), with one stage of K, with as many as its ring has and with more; rows of Y 16-byte aligned and not
@pytest.mark.parametrize("M,N,K,small", [(1, 1, 64, True), (129, 37, 128, True), (257, 136, 192, True), (300, 513, 448, True), (128, 128, 320, True),
                                         (1990, 3013, 64, False), (1990, 3016, 320, False), (2048, 4096, 192, False)])
@pytest.mark.parametrize("scaled", [False, True])
def test_gemm_dense(gpu_device, M, N, K, small, scaled):
    l = vq.lib()
    l._ZN2vq16gemm_dense_smallEii.restype = ctypes.c_bool
    assert l._ZN2vq16gemm_dense_smallEii(M, N) == small
    g = torch.Generator(device=gpu_device).manual_seed(4795 + M + K)
    X = torch.randn((M, K), generator=g, device=gpu_device).to(torch.float16)
    W = (torch.randn((N, K), generator=g, device=gpu_device) * 0.05).to(torch.float16)
    scale = (torch.rand(N, generator=g, device=gpu_device) + 0.5).to(torch.float16) if scaled else None
    Y = torch.full((M + 1, N), 7.0, dtype=torch.float16, device=gpu_device)
    ptr = lambda t: ctypes.c_void_p(0 if t is None else t.data_ptr())  # noqa: E731
    torch.cuda.synchronize()
    assert l._ZN2vq17launch_gemm_denseEPKDF16_S1_S1_PDF16_iiiP12ihipStream_t(ptr(X), ptr(W), ptr(scale), ptr(Y), M, N, K, ptr(None)) == 0
    torch.cuda.synchronize()
    want = X.double().cpu().numpy() @ W.double().cpu().numpy().T * (1 if scale is None else scale.double().cpu().numpy())
    assert_close(Y[:M], want, f"dense {M}x{N}x{K}")
    assert (Y[M] == 7).all()


def _product_in_pieces(X, W, scale):
    """X W^T in 64 bits on the GPU, over pieces of a very long K."""
    want = torch.zeros((X.shape[0], W.shape[0]), dtype=torch.float64, device=X.device)
    for k in range(0, X.shape[1], 1 << 18):
        want += X[:, k:k + (1 << 18)].double() @ W[:, k:k + (1 << 18)].double().t()
    return (want if scale is None else want * scale.double()).cpu().numpy()


# Both sides of K = 2^22, up to which the second stage has 32-bit offsets in a tile (256 rows of X are 2 GiB there), every kind of
# dequantization; 24 columns are a whole strip of the ordered weight and a narrower one.  (One or two codebooks take one pass up to 2^22.)
@pytest.mark.parametrize("K,v,bits,R,E", [(1 << 22, 8, 8, 3, 256), (1 << 22, 4, 16, 3, 300), ((1 << 22) + 64, 8, 8, 3, 256), ((1 << 22) + 64, 8, 16, 1, 5001),
                                          ((1 << 22) + 64, 4, 8, 2, 200)])
def test_gemm_two_stage_at_the_limit_of_its_offsets(gpu_device, K, v, bits, R, E):
    M, N = 257, 24
    one_pass = vq.lib()._ZN2vq13gemm_one_passEPK11vq_weight_ti
    one_pass.restype = ctypes.c_bool
    fits = vq.lib()._ZN2vq15gemm_tiles_fitsEi
    fits.restype = ctypes.c_bool
    g = torch.Generator(device=gpu_device).manual_seed(4797 + v)
    codes = torch.randint(0, E, (N, K // v, R), generator=g, device=gpu_device, dtype=torch.int32).to(torch.uint16 if bits == 16 else torch.uint8)
    w = vq.VQWeightDev(N, K, v, bits, codes, (torch.randn((R, E, v), generator=g, device=gpu_device) * 0.02).to(torch.float16),
                       (torch.rand(N, generator=g, device=gpu_device) + 0.5).to(torch.float16))
    assert not one_pass(ctypes.byref(w.desc()), M) and fits(K) == (K <= 1 << 22) and vq.vq_gemm_workspace(w, M) == N * K * 2
    X = torch.randn((M, K), generator=g, device=gpu_device, dtype=torch.float16)
    Y = vq.vq_gemm(w, X)
    assert_close(Y, _product_in_pieces(X, vq.vq_dequant(w, out_fp32=False), w.scale), f"K {K} v {v} R {R}")


# ... and the tiles with the longest offsets: 256 rows of X, and 256 columns of the weight
@pytest.mark.parametrize("pick,M,N", [(0, 256, 24), (1, 300, 72), (2, 128, 250)])
def test_gemm_tiles_at_the_limit_of_their_offsets(gpu_device, pick, M, N):
    K = 1 << 22
    g = torch.Generator(device=gpu_device).manual_seed(4799 + pick)
    X = torch.randn((M, K), generator=g, device=gpu_device, dtype=torch.float16)
    W = torch.randn((N, K), generator=g, device=gpu_device, dtype=torch.float16) * 0.02
    pieces = []     # operand order: strips of 16 columns, fragments of 32 k, groups of 8
    for n in range(0, N, 16):
        strip = W[n:n + 16]
        pieces.append(strip.view(strip.shape[0], K // 8, 8).transpose(0, 1).reshape(-1))
    ordered = torch.cat(pieces)
    Y = torch.full((M + 1, N), 7.0, dtype=torch.float16, device=gpu_device)
    ptr = lambda t: ctypes.c_void_p(0 if t is None else t.data_ptr())  # noqa: E731
    torch.cuda.synchronize()
    assert vq.lib()._ZN2vq17launch_gemm_tilesEPKDF16_S1_S1_PDF16_iiiiP12ihipStream_t(ptr(X), ptr(ordered), ptr(None), ptr(Y), M, N, K, pick, ptr(None)) == 0
    torch.cuda.synchronize()
    assert_close(Y[:M], _product_in_pieces(X, W, None), f"tile {pick} {M}x{N}x{K}")
    assert (Y[M] == 7).all()


# One pass over the codes for 17 .. 256 tokens: every tile of the kernel ({weight rows} x {tokens} of a workgroup: 16 x 16,
# 16 x 32, 32 x 32, 32 x 64, 64 x 64 from LDS; 16 x 16 .. 32 x 128 from L2) at ragged N, M and K, several iterations per
# wavefront among them.  Codes are in range, so the bound is that of the other products (fp16 operands, fp32 sums).
@pytest.mark.parametrize("N,K,M", [(33, 64, 17), (37, 1216, 18), (20, 2304, 256), (2051, 192, 17), (2051, 320, 33), (4099, 192, 33),
                                   (8195, 64, 17), (8200, 320, 63), (131, 320, 401)])
@pytest.mark.parametrize("v,bits,R,E", [(8, 8, 1, 256), (8, 8, 2, 200), (4, 8, 1, 256), (4, 8, 2, 256), (8, 12, 2, 4096), (8, 12, 1, 4096),
                                        (4, 12, 2, 512), (8, 16, 2, 2048), (4, 16, 1, 1000), (4, 16, 2, 256)])
def test_gemm_skinny_lds_codebooks(gpu_device, N, K, M, v, bits, R, E):
    w = wl.make_weight(N, K, v, bits, R, E, 0.02 / R, seed=4800 + N + K, with_scale=(N + R) % 2 == 0)
    X = wl.make_activations(M, K, seed=4801 + M)
    Y = vq.vq_gemm(vq.weight_to_device(w, gpu_device), dev_x(X, gpu_device))
    assert_close(Y, oracle.gemm(ocodes(w), w.codebooks, w.scale, X), f"skinny gemm {M}x{N}x{K} v{v} b{bits} R{R}")


@pytest.mark.parametrize("v", [8, 4])
@pytest.mark.parametrize("N,K,M", [(33, 64, 17), (37, 1216, 2), (64, 8320, 5), (1500, 192, 17), (1500, 320, 33), (1029, 64, 129),
                                   (2051, 192, 129), (4099, 64, 17), (515, 1024, 256), (130, 320, 8), (130, 320, 16), (131, 320, 401)])
def test_gemm_skinny_l2_codebook(gpu_device, N, K, M, v):
    w = wl.make_weight(N, K, v, 16, 1, 65536, 0.02, seed=4850 + N + K, with_scale=N % 2 == 1)
    X = wl.make_activations(M, K, seed=4851 + M)
    wd = vq.weight_to_device(w, gpu_device)
    Y = vq.vq_gemm(wd, dev_x(X, gpu_device)) if M > 16 else vq.vq_gemv(wd, dev_x(X, gpu_device))
    assert_close(Y, oracle.gemm(w.codes, w.codebooks, w.scale, X), f"skinny gemm {M}x{N}x{K} v{v} 2^16")


# more than 256 tokens where the two-stage product does not exist (K % 64 == 32)
@pytest.mark.parametrize("N,K,M", [(130, 96, 257), (37, 1248, 300), (515, 4128, 1025)])
@pytest.mark.parametrize("v,bits,R,E", [(8, 12, 2, 4096), (4, 16, 1, 65536), (4, 8, 2, 256), (8, 16, 2, 2048)])
def test_gemm_skinny_many_tokens_half_a_block_of_k(gpu_device, N, K, M, v, bits, R, E):
    w = wl.make_weight(N, K, v, bits, R, E, 0.02 / R, seed=4880 + N + K)
    X = wl.make_activations(M, K, seed=4881 + M)
    Y = vq.vq_gemm(vq.weight_to_device(w, gpu_device), dev_x(X, gpu_device))
    assert_close(Y, oracle.gemm(ocodes(w), w.codebooks, w.scale, X), f"skinny gemm {M}x{N}x{K} v{v} b{bits} R{R}")


# tiles of 48 tokens, with one and with two row tiles: their edges, ragged N and K, every format
@pytest.mark.parametrize("N,K,M", [(33, 192, 33), (4100, 192, 48), (4100, 1216, 65), (2051, 320, 96), (1000, 2304, 140), (8200, 448, 47)])
@pytest.mark.parametrize("v,bits,R,E", [(8, 8, 1, 256), (8, 8, 2, 200), (4, 8, 1, 256), (4, 8, 2, 100), (8, 12, 2, 1000), (8, 12, 1, 4096), (8, 16, 1, 4096), (4, 16, 2, 900)])
def test_gemm_skinny_48_tokens(gpu_device, N, K, M, v, bits, R, E):
    w = wl.make_weight(N, K, v, bits, R, E, 0.02 / R, seed=4990 + N + M)
    X = wl.make_activations(M, K, seed=4991 + M)
    Y = vq.vq_gemm(vq.weight_to_device(w, gpu_device), dev_x(X, gpu_device))
    assert_close(Y, oracle.gemm(ocodes(w), w.codebooks, w.scale, X), f"skinny gemm {M}x{N}x{K} v{v} b{bits} R{R}")


def test_gemm_skinny_x_beyond_32_bit_offsets(gpu_device):
    # 513 tokens of K = 2^22 - 32: byte offsets into X fit 32 bits for 512 tokens, so the last one goes in a second launch
    N, K, M = 16, (1 << 22) - 32, 513
    g = torch.Generator(device=gpu_device)
    g.manual_seed(4895)
    codes = torch.randint(0, 256, (N, K // 4, 2), generator=g, device=gpu_device, dtype=torch.uint8)
    cb = (torch.randn((2, 256, 4), generator=g, device=gpu_device) * 0.001).to(torch.float16)
    w = vq.VQWeightDev(N, K, 4, 8, codes, cb, None)
    X = torch.randn((M, K), generator=g, device=gpu_device, dtype=torch.float16)
    Y = vq.vq_gemm(w, X).double().cpu().numpy()
    W = vq.vq_dequant(w, out_fp32=False).float()
    for m in (0, 255, 511, 512):
        want = (W * X[m].float()).sum(1, dtype=torch.float64).cpu().numpy()
        assert np.linalg.norm(Y[m] - want) <= 2e-3 * np.linalg.norm(want), m


@pytest.mark.parametrize("E", [1, 1001, 16383])      # odd: no whole 16-byte pieces, so not staged in LDS
@pytest.mark.parametrize("N,K,M", [(37, 1216, 18), (1500, 320, 33), (2051, 192, 129), (515, 1024, 256), (131, 320, 401)])
def test_gemm_skinny_odd_codebook(gpu_device, N, K, M, E):
    w = wl.make_weight(N, K, 4, 16, 1, E, 0.02, seed=4870 + N + E, with_scale=N % 2 == 1)
    X = wl.make_activations(M, K, seed=4871 + M)
    Y = vq.vq_gemm(vq.weight_to_device(w, gpu_device), dev_x(X, gpu_device))
    assert_close(Y, oracle.gemm(w.codes, w.codebooks, w.scale, X), f"skinny gemm {M}x{N}x{K} v4 E{E}")


@pytest.mark.parametrize("bits,E,M", [(8, 256, 20), (16, 65536, 20), (16, 65536, 3)])
def test_gemm_skinny_infinities_at_the_end_of_a_row(gpu_device, bits, E, M):
    # K = 192 leaves half of an iteration past the end of every row; there the last codes and activations are read again,
    # and an infinity among them must not meet a zero
    w = wl.make_weight(40, 192, 8, bits, 1, E, 0.02, seed=4890, with_scale=False)
    w.codes[:, -1, 0] = 7
    w.codes[:, :-1, 0][w.codes[:, :-1, 0] == 7] = 8
    w.codebooks[0, 7] = np.float16(0.01)
    X = wl.make_activations(M, 192, seed=4891)
    X[1, -1] = np.float16(np.inf)
    wd = vq.weight_to_device(w, gpu_device)
    Y = (vq.vq_gemm(wd, dev_x(X, gpu_device)) if M > 16 else vq.vq_gemv(wd, dev_x(X, gpu_device))).float().cpu().numpy()
    assert np.isposinf(Y[1]).all()
    rest = np.delete(np.arange(M), 1)
    assert_close(torch.from_numpy(Y[rest]), oracle.gemm(w.codes, w.codebooks, None, X[rest]), "other tokens")


def test_gemm_rows_match_gemv(gpu_device):
    # the prefill product of a few tokens and the decode product of the same tokens agree to tolerance
    w = wl.make_weight(256, 1024, 8, 16, 1, 65536, 0.02, seed=4600)
    X = wl.make_activations(64, 1024, seed=4601)
    wd = vq.weight_to_device(w, gpu_device)
    Y = vq.vq_gemm(wd, dev_x(X, gpu_device)).float().cpu().numpy()
    y = vq.vq_gemv(wd, dev_x(X[:16].copy(), gpu_device)).float().cpu().numpy()
    assert np.linalg.norm(Y[:16] - y) / np.linalg.norm(y) < 1e-3


# ---------------------------------------------------------------- VQ-attn decode

def run_attn(kv, device, sm_scale):
    kd = vq.kv_to_device(kv, device)
    out = vq.vq_attn_decode(kd, dev_x(kv.q, device), sm_scale)
    torch.cuda.synchronize()
    return out


def oracle_attn(kv, sm_scale):
    return oracle.attn_decode(kv.k_codes, kv.v_codes, kv.k_codebooks, kv.v_codebooks, kv.q, sm_scale,
                              seq_lens=kv.seq_lens)


@pytest.mark.parametrize("B,H,T,v,G,ragged", [
    (2, 3, 1, 4, 1, False),        # a single token: out = V[0]
    (2, 3, 300, 4, 1, False),
    (3, 2, 2048, 4, 1, True),      # exactly one token range, ragged lengths
    (2, 2, 2049, 4, 1, False),     # one token spills into a second range
    (2, 2, 5000, 4, 1, True),      # three ranges, ragged
    (1, 2, 700, 4, 32, False),     # one codebook per sub-space (coupled-quantization layout)
    (1, 2, 700, 4, 4, True),
    (1, 2, 513, 8, 1, False),
    (1, 2, 513, 8, 16, False),
    (1, 2, 513, 2, 1, True),
    (1, 2, 513, 2, 64, False),
])
def test_attn_small_full_compare(gpu_device, B, H, T, v, G, ragged):
    kv = wl.make_kv(B, H, 128, T, v, 256, G, seed=5000 + T + G + v, ragged=ragged)
    sm = 1.0 / np.sqrt(128.0)
    assert_close(run_attn(kv, gpu_device, sm), oracle_attn(kv, sm), f"attn B{B} H{H} T{T} v{v} G{G}")


# v = 4: one codebook per head, and 32 codebooks with one (T 1500) and two items per workgroup; odd numbers of items and of token
# ranges, one and two tokens past a 32-token unit, flat and sharp softmax (weights from 1 down to far below the smallest
# half), and a V codebook with an infinity that one token uses and a NaN that none does.
@pytest.mark.parametrize("sharp", [1.0, 6.0])
@pytest.mark.parametrize("B,H,T,G", [(13, 32, 33, 1), (16, 24, 290, 1), (3, 32, 1500, 32), (9, 32, 97, 32), (3, 32, 2050, 32)])
def test_attn_matrix_core_values(gpu_device, B, H, T, G, sharp):
    kv = wl.make_kv(B, H, 128, T, 4, 256, G, seed=5300 + T, ragged=sharp > 1)
    kv.q = (kv.q * np.float16(sharp)).astype(np.float16)
    sm = 1.0 / np.sqrt(128.0)
    assert_close(run_attn(kv, gpu_device, sm), oracle_attn(kv, sm), f"attn B{B} H{H} T{T} G{G} x{sharp}")


@pytest.mark.parametrize("B,H,T,G", [(16, 24, 290, 1), (3, 32, 1500, 32), (3, 32, 2050, 32), (16, 32, 4096, 1)])
def test_attn_matrix_core_values_with_infinities(gpu_device, B, H, T, G):
    kv = wl.make_kv(B, H, 128, T, 4, 256, G, seed=5350 + T)
    kv.v_codes[kv.v_codes == 7] = 8
    kv.v_codes[kv.v_codes == 9] = 8
    kv.v_codebooks[3, 0, 7, 1] = np.float16(-np.inf)      # element 1 of entry 7, head 3
    kv.v_codebooks[5, 0, 9, 2] = np.float16(np.nan)       # an entry that no token uses
    kv.v_codes[1, 3, T - 20, 0] = 7                       # channel 1 of batch entry 1, head 3
    want = oracle_attn(kv, 1.0 / np.sqrt(128.0))
    got = run_attn(kv, gpu_device, 1.0 / np.sqrt(128.0)).float().cpu().numpy()
    assert want[1, 3, 1] == -np.inf and got[1, 3, 1] == -np.inf
    want[1, 3, 1] = got[1, 3, 1] = 0
    assert_close(torch.from_numpy(got), want, "all other channels")


@pytest.mark.parametrize("B,H,T,G", [(16, 24, 290, 1), (9, 32, 97, 32), (3, 32, 2050, 32)])
@pytest.mark.parametrize("bits", [20, 30, 34, 38])
def test_attn_small_weights_of_large_values(gpu_device, B, H, T, G, bits):
    """In every run of 32 tokens one takes nearly all of the softmax and holds zeros in every fourth channel; the others
    have weights of 2^-bits and hold 60000 there, so those channels are sums of the small weights alone.  A weight is fp32 and
    may be off by the rounding of its exponent's argument (about 2^6, to 24 bits: 2^-18); the output by one rounding to half."""
    kv = wl.make_kv(B, H, 128, T, 4, 256, G, seed=5380 + T)
    sm = 1.0 / np.sqrt(128.0)
    kv.q[:] = 1
    kv.k_codes[:], kv.v_codes[:] = 1, 1
    kv.k_codes[:, :, 7::32], kv.v_codes[:, :, 7::32] = 0, 0
    kv.k_codebooks[:, :, 0], kv.k_codebooks[:, :, 1] = 0, np.float16(-bits * np.log(2.0) / (128 * sm))
    kv.v_codebooks[:, :, 0], kv.v_codebooks[:, :, 1] = np.float16([0, 0.5, -1, 2]), np.float16([60000, 1, 3, -2])
    want = oracle_attn(kv, sm)
    got = run_attn(kv, gpu_device, sm).double().cpu().numpy()
    bound = (2.0 ** -11 + 2.0 ** -17) * np.abs(want) + 2.0 ** -25
    assert (np.abs(got - want) <= bound).all(), (want[0, 0, 0], got[0, 0, 0])


def test_attn_two_sequences_per_workgroup_odd_batch_and_empty_sequences(gpu_device):
    # 32 codebooks per head and side: pairs of batch entries share a workgroup; the batch is odd, one
    # sequence is empty and one stops inside the first token range while its partner goes on
    kv = wl.make_kv(5, 2, 128, 1300, 4, 256, 32, seed=5200)
    kv.seq_lens = np.array([1300, 0, 37, 1300, 600], dtype=np.int32)
    sm = 1.0 / np.sqrt(128.0)
    out = run_attn(kv, gpu_device, sm)
    assert (out[1] == 0).all()
    assert_close(out, oracle_attn(kv, sm), "attn pairs")


@pytest.mark.parametrize("B,H,T,E,lens", [
    (3, 64, 1000, 256, [1000, 0, 513]),      # odd batch, an empty sequence, two token ranges per sequence
    (4, 96, 300, 256, None),                 # one range, 192 workgroups
    (2, 256, 77, 200, [77, 5]),              # fewer entries than 256, a single ragged tile
])
def test_attn_replicated_codebooks(gpu_device, B, H, T, E, lens):
    """One codebook per head and side and enough workgroups for one per compute unit, but ranges too short for copies of the
    codebook in LDS (those: the test below)."""
    kv = wl.make_kv(B, H, 128, T, 4, E, 1, seed=5300 + B + H)
    if lens is not None:
        kv.seq_lens = np.array(lens, dtype=np.int32)
    sm = 1.0 / np.sqrt(128.0)
    out = run_attn(kv, gpu_device, sm)
    assert_close(out, oracle_attn(kv, sm), f"attn replicated B{B} H{H} T{T}")
    assert torch.equal(out, run_attn(kv, gpu_device, sm))
    if lens is not None and 0 in lens:
        assert (out[lens.index(0)] == 0).all()


# Shapes at which the copies are used: one and two ranges per sequence, an odd number of items; most sequences short or empty
@pytest.mark.parametrize("B,H,T,lens", [(16, 32, 4096, [4096, 0, 1, 33, 300, 31]), (8, 32, 8192, [5000, 0, 4097, 70]), (33, 30, 4096, [1500, 64, 0, 7])])
def test_attn_replicated_codebooks_of_long_ranges(gpu_device, B, H, T, lens):
    kv = wl.make_kv(B, H, 128, T, 4, 250, 1, seed=7150 + B)
    kv.seq_lens = np.array([lens[b] if b < len(lens) else 0 for b in range(B - 1)] + [200], dtype=np.int32)
    kd = vq.kv_to_device(kv, gpu_device)
    assert vq.lib()._ZN2vq15attn_replicatedEPK7vq_kv_t(ctypes.byref(kd.desc())) & 0xFF
    sm = 1.0 / np.sqrt(128.0)
    out = vq.vq_attn_decode(kd, dev_x(kv.q, gpu_device), sm)
    torch.cuda.synchronize()
    assert_close(out, oracle_attn(kv, sm), f"attn replicated B{B} H{H} T{T}")
    assert (out[1 if lens[1] == 0 else 2] == 0).all()


def test_attn_zero_length_sequence_and_sharp_softmax(gpu_device):
    kv = wl.make_kv(3, 2, 128, 600, 4, 256, 1, seed=5100)
    kv.seq_lens = np.array([600, 0, 1], dtype=np.int32)
    sm = 1.0                                  # un-scaled scores ~ N(0, 128): nearly one-hot softmax
    out = run_attn(kv, gpu_device, sm)
    want = oracle_attn(kv, sm)
    assert (out[1] == 0).all()
    assert_close(out, want, "attn len0 / sharp")


def test_attn_config5_coupled_quantization_layout_full_size(gpu_device):
    # the paper's CQ-2 layout (Sec. III-B, Tbl. IV): one codebook per 4-channel sub-space, 32 per head and
    # side (64 KiB of K codebooks per head), at the full C5 shape
    kv = wl.config5_kv(G=32)
    sm = 1.0 / np.sqrt(128.0)
    out = run_attn(kv, gpu_device, sm)
    assert_close(out, oracle_attn(kv, sm), "C5 G=32 full")


@pytest.mark.parametrize("B,H,T,v,G,ragged", [
    (2, 3, 1, 4, 32, False),       # a single token
    (2, 2, 300, 4, 32, False),     # one partial range of 256 tokens + a tail
    (3, 2, 1000, 4, 32, True),     # ragged lengths (with a full-length sequence)
    (2, 2, 513, 2, 64, False),     # CQ-4: 16 codes per channel group and token
    (1, 2, 700, 8, 16, True),      # v = 8: 4 codes per channel group
    (2, 2, 400, 4, 4, False),      # one codebook per channel group (the coarsest layout the variant takes)
])
def test_attn_channel_parallel(gpu_device, B, H, T, v, G, ragged):
    """vq_attn_decode_channel_parallel (Sec. VI-A codebook-centric dataflow with global accumulation of the partial
    inner products) against the oracle and against the token-parallel kernel; repeated calls bit-identical."""
    kv = wl.make_kv(B, H, 128, T, v, 256, G, seed=8800 + T + G, ragged=ragged)
    if ragged:
        kv.seq_lens[-1] = 0                              # an empty sequence yields zeros
    sm = 1.0 / np.sqrt(128.0)
    kd = vq.kv_to_device(kv, gpu_device)
    qd = dev_x(kv.q, gpu_device)
    out = vq.vq_attn_decode_channel_parallel(kd, qd, sm)
    torch.cuda.synchronize()
    want = oracle_attn(kv, sm)
    assert_close(out, want, "channel-parallel")
    assert_close(vq.vq_attn_decode(kd, qd, sm), want, "token-parallel, same cache")
    again = vq.vq_attn_decode_channel_parallel(kd, qd, sm)
    torch.cuda.synchronize()
    assert torch.equal(out, again)
    if ragged:
        assert float(out[-1].abs().max()) == 0.0


def test_attn_channel_parallel_config5_cq_full_size(gpu_device):
    kv = wl.config5_kv(G=32)
    sm = 1.0 / np.sqrt(128.0)
    kd = vq.kv_to_device(kv, gpu_device)
    out = vq.vq_attn_decode_channel_parallel(kd, dev_x(kv.q, gpu_device), sm)
    torch.cuda.synchronize()
    assert_close(out, oracle_attn(kv, sm), "C5 G=32 full, channel-parallel")


def test_attn_config5_cq4_full_size(gpu_device):
    # the paper's CQ-4 row (Tbl. III: VQ<2,8,1>): one codebook per 2-channel sub-space, 64 per head and side
    # (64 KiB of K codebooks per head), 64 code bytes per token and side, at the full C5 shape
    kv = wl.config5_kv(G=64, v=2)
    sm = 1.0 / np.sqrt(128.0)
    out = run_attn(kv, gpu_device, sm)
    assert_close(out, oracle_attn(kv, sm), "C5 CQ-4 full")


def test_attn_config5_full_size(gpu_device):
    kv = wl.config5_kv()
    sm = 1.0 / np.sqrt(128.0)
    out = run_attn(kv, gpu_device, sm)
    assert_close(out, oracle_attn(kv, sm), "C5 full")
    again = run_attn(kv, gpu_device, sm)
    assert torch.equal(out, again)            # fixed-order reductions: bit-identical repeats


# ---------------------------------------------------------------- per-tile codebooks (Sec. III-B, Tbl. III)

def run_dequant_tiled(w, device, fp32):
    wd = vq.weight_to_device(w, device)
    out = vq.vq_dequant(wd, out_fp32=fp32)
    torch.cuda.synchronize()
    return out


@pytest.mark.parametrize("N,K,v,bits,R,E,tile", [
    (512, 512, 4, 8, 1, 256, (256, 256)),     # the paper's per-tile row: VQ<4,8,1>, (256, 256) tiles
    (300, 384, 8, 8, 2, 64, (64, 128)),       # ragged last row tile, residual codebooks
    (96, 256, 8, 16, 1, 1024, (32, 64)),      # uint16 codes
])
def test_per_tile_codebooks_dequant_and_gemv(gpu_device, N, K, v, bits, R, E, tile):
    w = wl.make_weight(N, K, v, bits, R, E, 0.02, seed=8100 + N, cb_tile=tile)
    want32 = oracle.dequant(w.codes, w.codebooks, cb_tile=tile)
    got32 = run_dequant_tiled(w, gpu_device, True).cpu().numpy()
    assert got32.tobytes() == want32.tobytes()                              # bit-exact fp32 tiles
    got16 = run_dequant_tiled(w, gpu_device, False).cpu().numpy()
    assert got16.tobytes() == want32.astype(np.float16).tobytes()          # and their fp16 rounding
    for bs in (1, 7, 16):
        x = wl.make_activations(bs, K, 8200 + bs)
        assert_close(run_gemv(w, x, gpu_device), oracle.gemv(w.codes, w.codebooks, w.scale, x, cb_tile=tile),
                     f"tiled gemv bs{bs}")


def test_per_tile_codebooks_full_size_gemv_and_gemm(gpu_device):
    w = wl.gptvq_like_layer(1)                                              # 11008 x 4096, 43 x 16 tiles
    x = wl.make_activations(1, w.K, 8300)
    assert_close(run_gemv(w, x, gpu_device), oracle.gemv(w.codes, w.codebooks, w.scale, x, cb_tile=w.cb_tile),
                 "tiled gemv full")
    X = wl.make_activations(300, w.K, 8301)                                 # two-stage prefill path (M > 256)
    rows = np.arange(0, w.N, 97)
    wd = vq.weight_to_device(w, gpu_device)
    Y = vq.vq_gemm(wd, dev_x(X, gpu_device))
    torch.cuda.synchronize()
    want = oracle.gemm(w.codes, w.codebooks, w.scale, X, rows=rows, cb_tile=w.cb_tile)
    assert_close(Y[:, torch.from_numpy(rows).to(gpu_device)], want, "tiled gemm")
    Ys = vq.vq_gemm(wd, dev_x(X[:40], gpu_device))                          # small M: goes through the gemv kernels
    torch.cuda.synchronize()
    assert_close(Ys[:, torch.from_numpy(rows).to(gpu_device)], want[:40], "tiled gemm small M")


# ---------------------------------------------------------------- packed 12-bit codes (VQ<8,12,2>, Sec. VII-B)

def ocodes(w):
    """The codes of a host weight as the oracle takes them."""
    if w.code_bits == 12:
        return oracle.Packed12(w.codes, (w.N, w.K // w.v, w.R))
    return w.codes


@pytest.mark.parametrize("N,K,v,R,E", [
    (200, 512, 8, 2, 4096),      # the paper's configuration: two additive 4096-entry codebooks
    (96, 256, 8, 1, 3000),       # one codebook, E below the 12-bit range
    (64, 128, 4, 4, 512),        # v = 4, four residual codebooks
])
def test_packed_12_bit_codes_dequant_gemv_gemm(gpu_device, N, K, v, R, E):
    w = wl.make_weight(N, K, v, 12, R, E, 0.01, seed=8500 + N)
    want32 = oracle.dequant(ocodes(w), w.codebooks)
    wd = vq.weight_to_device(w, gpu_device)
    got32 = vq.vq_dequant(wd, out_fp32=True)
    torch.cuda.synchronize()
    assert got32.cpu().numpy().tobytes() == want32.tobytes()                # bit-exact tiles
    for bs in (1, 9, 16):
        x = wl.make_activations(bs, K, 8600 + bs)
        assert_close(vq.vq_gemv(wd, dev_x(x, gpu_device)), oracle.gemv(ocodes(w), w.codebooks, w.scale, x),
                     f"12-bit gemv bs{bs}")
    X = wl.make_activations(300, K, 8700)
    assert_close(vq.vq_gemm(wd, dev_x(X, gpu_device)), oracle.gemm(ocodes(w), w.codebooks, w.scale, X), "12-bit gemm")


def test_packed_12_bit_full_size(gpu_device):
    w = wl.aqlm3_like_layer(0)                                               # 4096 x 4096, 128 KiB of codebooks
    x = wl.make_activations(4, w.K, 8800)
    wd = vq.weight_to_device(w, gpu_device)
    assert_close(vq.vq_gemv(wd, dev_x(x, gpu_device)), oracle.gemv(ocodes(w), w.codebooks, w.scale, x), "AQLM-3-like gemv")


# ---------------------------------------------------------------- on-the-fly KV quantization (Sec. II-A, Sec. VII)

@pytest.mark.parametrize("B,H,T,v,G,n_new,pos", [
    (2, 3, 40, 4, 1, 1, 39),        # decode: one new token at the end of the cache
    (2, 2, 300, 4, 32, 130, 7),     # prefill chunk, one codebook per sub-space, several token chunks
    (1, 2, 64, 8, 4, 64, 0),
    (1, 2, 50, 2, 1, 5, 20),
    (3, 5, 33, 8, 1, 1, 32),        # decode, v = 8: 16 items per side, 16 lanes each
    (2, 3, 20, 2, 1, 2, 3),         # two new tokens, v = 2: 128 items per side
    (2, 2, 16, 4, 32, 1, 15),       # decode with one codebook per sub-space (sides staged one after the other)
])
def test_kv_quantize_codes_bit_exact_and_in_place(gpu_device, B, H, T, v, G, n_new, pos):
    kv = wl.make_kv(B, H, 128, T, v, 256, G, seed=9300 + T)
    rng = np.random.default_rng(9301 + T)
    k_new = rng.normal(0, 1, size=(B, H, n_new, 128)).astype(np.float16)
    v_new = rng.normal(0, 1, size=(B, H, n_new, 128)).astype(np.float16)
    kd = vq.kv_to_device(kv, gpu_device)
    vq.vq_kv_quantize(kd, dev_x(k_new, gpu_device), dev_x(v_new, gpu_device), pos)
    torch.cuda.synchronize()
    want_k, want_v = kv.k_codes.copy(), kv.v_codes.copy()
    want_k[:, :, pos:pos + n_new] = oracle.kv_quantize(k_new, kv.k_codebooks)
    want_v[:, :, pos:pos + n_new] = oracle.kv_quantize(v_new, kv.v_codebooks)
    assert np.array_equal(kd.k_codes.cpu().numpy(), want_k)          # integer result: exact; the rest untouched
    assert np.array_equal(kd.v_codes.cpu().numpy(), want_v)


def test_kv_quantize_ties_go_to_the_smallest_index(gpu_device):
    # a codebook of four distinct entries repeated 64 times: every sub-vector has 64 equally close entries,
    # spread over all the lanes that share the item; the smallest index must win (decode and prefill paths)
    for n_new in (1, 70):
        kv = wl.make_kv(2, 2, 128, 80, 4, 256, 1, seed=9100 + n_new)
        for cb in (kv.k_codebooks, kv.v_codebooks):
            cb[:] = np.tile(cb[:, :, :4, :], (1, 1, 64, 1))
        rng = np.random.Generator(np.random.PCG64(9101))
        k_new = rng.normal(0, 1, size=(2, 2, n_new, 128)).astype(np.float16)
        v_new = rng.normal(0, 1, size=(2, 2, n_new, 128)).astype(np.float16)
        kd = vq.kv_to_device(kv, gpu_device)
        vq.vq_kv_quantize(kd, dev_x(k_new, gpu_device), dev_x(v_new, gpu_device), 5)
        torch.cuda.synchronize()
        got_k = kd.k_codes.cpu().numpy()[:, :, 5:5 + n_new]
        got_v = kd.v_codes.cpu().numpy()[:, :, 5:5 + n_new]
        assert got_k.max() < 4 and got_v.max() < 4
        assert np.array_equal(got_k, oracle.kv_quantize(k_new, kv.k_codebooks))
        assert np.array_equal(got_v, oracle.kv_quantize(v_new, kv.v_codebooks))


@pytest.mark.parametrize("v,G,E,n_new", [(4, 1, 256, 5), (4, 1, 256, 6), (4, 32, 250, 17), (2, 64, 256, 129), (8, 2, 33, 40), (4, 1, 8, 300),
                                          (4, 1, 30, 70), (8, 2, 10, 40), (2, 64, 60, 40), (4, 32, 120, 40)])
@pytest.mark.parametrize("kind", ["plain", "near_ties", "tiny", "huge", "not_finite"])
def test_kv_quantize_hard_values(gpu_device, v, G, E, n_new, kind):
    """The matrix-core kernel rules entries out by an approximate distance: entries that differ in the last bits, codebooks
    whose squares leave the range of its scaled halves, and values that are not finite must give the definition's codes."""
    kv = wl.make_kv(1, 2, 128, n_new + 3, v, E, G, seed=9500 + E + n_new)
    rng = np.random.default_rng(9501 + E + n_new)
    x = rng.normal(0, 1, size=(2, 1, 2, n_new, 128)).astype(np.float16)
    for cb in (kv.k_codebooks, kv.v_codebooks):
        if kind == "near_ties":   # copies of a few entries, one unit in the last place apart
            cb[:] = np.resize(cb[:, :, :max(1, E // 8), :], cb.shape)
            bits = cb.view(np.uint16)
            bits[:, :, ::3, 0] += 1
        elif kind == "tiny":
            cb *= np.float16(2.0 ** -13)
        elif kind == "huge":
            cb *= np.float16(12000.0)
        elif kind == "not_finite":
            cb[0, 0, E // 2, 0] = np.inf
            x[:, 0, 0, 1, :8] = np.inf
            x[:, 0, 0, 2, 8:16] = np.nan
    if kind == "tiny":
        x *= np.float16(2.0 ** -13)
    elif kind == "huge":
        x *= np.float16(12000.0)
    kd = vq.kv_to_device(kv, gpu_device)
    vq.vq_kv_quantize(kd, dev_x(x[0], gpu_device), dev_x(x[1], gpu_device), 2)
    torch.cuda.synchronize()
    assert np.array_equal(kd.k_codes.cpu().numpy()[:, :, 2:2 + n_new], oracle.kv_quantize(x[0], kv.k_codebooks))
    assert np.array_equal(kd.v_codes.cpu().numpy()[:, :, 2:2 + n_new], oracle.kv_quantize(x[1], kv.v_codebooks))


# Few sequences: the scan (D = 8, and few tokens) and the matrix cores with 16 tokens per workgroup, 32 items at a time or 64 with norms:
# edges of the units, and near ties inside and between groups of eight entries (more tokens per workgroup: the test after this one)
@pytest.mark.parametrize("D,v,G,E", [(8, 8, 1, 256), (8, 8, 1, 250), (128, 4, 1, 256), (128, 4, 1, 240), (128, 2, 1, 256), (128, 4, 32, 256), (128, 8, 16, 64)])
@pytest.mark.parametrize("n_new", [4, 33, 64, 129, 161])
@pytest.mark.parametrize("apart", [0, 1, 8, 16])
def test_kv_quantize_units_and_near_ties(gpu_device, D, v, G, E, n_new, apart):
    rng = np.random.default_rng(9550 + E + n_new + apart)
    B, H, T, P = 1, 2, n_new + 3, D // v
    cb = rng.normal(0, 1, size=(2, H, G, E, v)).astype(np.float16)
    if apart:   # every entry of an even block of that length has a twin `apart` further on, in part one unit in the last place off
        for e in range(E - apart):
            if (e // apart) % 2 == 0:
                cb[:, :, :, e + apart] = cb[:, :, :, e]
        cb.view(np.uint16)[:, :, :, ::3, 0] += 1
    x = rng.normal(0, 1, size=(2, B, H, n_new, D)).astype(np.float16)
    codes = [torch.full((B, H, T, P), 255, dtype=torch.uint8, device=gpu_device) for _ in range(2)]
    kd = vq.VQKVDev(B, H, D, T, v, codes[0], codes[1], dev_x(cb[0], gpu_device), dev_x(cb[1], gpu_device))
    vq.vq_kv_quantize(kd, dev_x(x[0], gpu_device), dev_x(x[1], gpu_device), 2)
    torch.cuda.synchronize()
    for side in range(2):
        got = codes[side].cpu().numpy()
        assert np.array_equal(got[:, :, 2:2 + n_new], oracle.kv_quantize(x[side], cb[side])), side
        assert (got[:, :, :2] == 255).all() and (got[:, :, 2 + n_new:] == 255).all(), side


def kv_plan(kd, n_new):
    """(kernel, way, tokens per workgroup, threads) of a call: what the library itself goes by."""
    out = (ctypes.c_int * 5)()
    vq.lib()._ZN2vq19kv_quantize_plan_ofEPK7vq_kv_tiPi(ctypes.byref(kd.desc()), n_new, out)
    return ("scan", "lane", "matrix")[out[0]], ("pair", "own", "norms")[out[1]], out[2], out[3]


# The matrix-core kernel by every way of looking at the best group of entries (two lanes per item, each lane its own item by the
# definition's distances, the same by norms), every number of tiles of entries, up to 128 tokens per workgroup with one that is not full,
# and both numbers of wavefronts; what is meant is asserted.  With twins of entries 8 further on, and without.
@pytest.mark.parametrize("apart", [0, 8])
@pytest.mark.parametrize("B,H,D,v,G,E,n_new,way,tokens,threads", [
    (2, 32, 128, 4, 1, 256, 1025, "norms", 128, 256), (2, 32, 128, 4, 1, 240, 1090, "norms", 128, 256), (2, 32, 128, 2, 1, 256, 1027, "norms", 128, 256),
    (2, 32, 128, 4, 1, 250, 1100, "own", 128, 256), (2, 32, 128, 8, 1, 256, 1033, "norms", 128, 256), (4, 32, 64, 8, 1, 201, 640, "own", 128, 256),
    (2, 32, 128, 4, 32, 256, 1031, "own", 128, 512), (2, 32, 128, 2, 64, 256, 1026, "own", 128, 512), (2, 32, 128, 8, 16, 256, 1040, "own", 128, 512),
    (2, 32, 256, 4, 1, 256, 1030, "norms", 128, 256), (2, 32, 128, 4, 1, 250, 513, "own", 64, 256), (1, 2, 128, 4, 1, 250, 33, "own", 16, 256),
    (1, 2, 128, 4, 1, 250, 129, "own", 16, 256), (2, 32, 128, 4, 1, 128, 1025, "norms", 128, 256), (2, 32, 128, 4, 1, 100, 1025, "own", 128, 256),
    (2, 32, 128, 4, 1, 64, 1025, "norms", 128, 256), (2, 32, 128, 4, 1, 50, 1025, "own", 128, 256), (16, 32, 64, 8, 8, 32, 300, "norms", 128, 256),
    (2, 32, 128, 8, 16, 64, 600, "norms", 64, 256), (1, 2, 128, 4, 32, 250, 33, "pair", 16, 512), (1, 8, 128, 8, 16, 100, 40, "pair", 16, 256), (2, 32, 128, 8, 1, 32, 1029, "norms", 128, 256),
])
def test_kv_quantize_prompts_by_every_way(gpu_device, B, H, D, v, G, E, n_new, way, tokens, threads, apart):
    rng = np.random.default_rng(9560 + E + n_new + apart)
    T, P = n_new + 3, D // v
    cb = rng.normal(0, 1, size=(2, H, G, E, v)).astype(np.float16)
    if apart:
        for e in range(E - apart):
            if (e // apart) % 2 == 0:
                cb[:, :, :, e + apart] = cb[:, :, :, e]
        cb.view(np.uint16)[:, :, :, ::3, 0] += 1
    g = torch.Generator(device=gpu_device).manual_seed(9570 + n_new)
    x = [torch.randn((B, H, n_new, D), generator=g, device=gpu_device).to(torch.float16) for _ in range(2)]
    codes = [torch.full((B, H, T, P), 255, dtype=torch.uint8, device=gpu_device) for _ in range(2)]
    kd = vq.VQKVDev(B, H, D, T, v, codes[0], codes[1], dev_x(cb[0], gpu_device), dev_x(cb[1], gpu_device))
    assert kv_plan(kd, n_new) == ("matrix", way, tokens, threads)
    vq.vq_kv_quantize(kd, x[0], x[1], 2)
    torch.cuda.synchronize()
    heads = [0, H // 2, H - 1]      # (the oracle takes its time)
    for side in range(2):
        got, xs = codes[side].cpu().numpy(), x[side][:, heads].contiguous().cpu().numpy()
        assert np.array_equal(got[:, heads, 2:2 + n_new], oracle.kv_quantize(xs, np.ascontiguousarray(cb[side][heads]))), side
        assert (got[:, :, :2] == 255).all() and (got[:, :, 2 + n_new:] == 255).all(), side


# head sizes other than 128: sub-vectors per group that are no power of two, one sub-vector per group, and the most LDS that
# staged codebooks take (D = 256: 128 KiB); a last workgroup that is not full
@pytest.mark.parametrize("D,v,G,E", [(96, 4, 1, 256), (96, 8, 4, 256), (80, 8, 2, 250), (192, 2, 32, 256), (40, 2, 5, 200), (24, 8, 3, 256),
                                     (8, 8, 1, 256), (256, 4, 1, 256), (256, 8, 32, 64), (256, 2, 128, 128),
                                     # fewer entries: one, two and four tiles of 32 with groups of eight that are partly or
                                     # wholly empty; a lane per sub-vector (E v <= 64)
                                     (128, 4, 1, 18), (128, 8, 2, 9), (96, 2, 16, 40), (128, 4, 1, 66), (128, 2, 64, 100), (128, 8, 4, 128),
                                     (128, 4, 1, 16), (96, 8, 12, 7), (256, 2, 128, 32), (128, 4, 32, 2), (40, 2, 5, 24), (128, 8, 1, 1)])
@pytest.mark.parametrize("n_new", [1, 3, 7, 300])
def test_kv_quantize_head_sizes(gpu_device, D, v, G, E, n_new):
    rng = np.random.default_rng(9600 + D + v + n_new)
    B, H, T, P = 1, 3, n_new + 5, D // v
    cb = rng.normal(0, 1, size=(2, H, G, E, v)).astype(np.float16)
    x = rng.normal(0, 1, size=(2, B, H, n_new, D)).astype(np.float16)
    codes = [torch.full((B, H, T, P), 255, dtype=torch.uint8, device=gpu_device) for _ in range(2)]
    kd = vq.VQKVDev(B, H, D, T, v, codes[0], codes[1], dev_x(cb[0], gpu_device), dev_x(cb[1], gpu_device))
    vq.vq_kv_quantize(kd, dev_x(x[0], gpu_device), dev_x(x[1], gpu_device), 4)
    torch.cuda.synchronize()
    for side in range(2):
        got = codes[side].cpu().numpy()
        assert np.array_equal(got[:, :, 4:4 + n_new], oracle.kv_quantize(x[side], cb[side])), side
        assert (got[:, :, :4] == 255).all() and (got[:, :, 4 + n_new:] == 255).all(), side


def test_kv_quantize_then_attend(gpu_device):
    # a cache written by the quantizer, read by the attention kernel: compare with the oracle's two steps
    B, H, T = 2, 4, 700
    kv = wl.make_kv(B, H, 128, T, 4, 256, 1, seed=9400)
    rng = np.random.default_rng(9401)
    # realistic new vectors: entries plus noise, so that the closest entry is usually clear
    k_all = (oracle.kv_dequant(kv.k_codes, kv.k_codebooks) + rng.normal(0, 0.05, size=(B, H, T, 128))).astype(np.float16)
    v_all = (oracle.kv_dequant(kv.v_codes, kv.v_codebooks) + rng.normal(0, 0.05, size=(B, H, T, 128))).astype(np.float16)
    kd = vq.kv_to_device(kv, gpu_device)
    kd.k_codes.zero_()
    kd.v_codes.zero_()
    vq.vq_kv_quantize(kd, dev_x(k_all[:, :, :650], gpu_device), dev_x(v_all[:, :, :650], gpu_device), 0)   # prefill
    for t in range(650, 700, 10):                                                                         # then decode steps
        vq.vq_kv_quantize(kd, dev_x(k_all[:, :, t:t + 10], gpu_device), dev_x(v_all[:, :, t:t + 10], gpu_device), t)
    sm = 1.0 / np.sqrt(128.0)
    out = vq.vq_attn_decode(kd, dev_x(kv.q, gpu_device), sm)
    torch.cuda.synchronize()
    kc, vc = oracle.kv_quantize(k_all, kv.k_codebooks), oracle.kv_quantize(v_all, kv.v_codebooks)
    assert np.array_equal(kd.k_codes.cpu().numpy(), kc) and np.array_equal(kd.v_codes.cpu().numpy(), vc)
    assert_close(out, oracle.attn_decode(kc, vc, kv.k_codebooks, kv.v_codebooks, kv.q, sm), "quantize + attend")


# ---------------------------------------------------------------- randomized sweep over formats and shapes

def _random_weight_case(rng):
    v = int(rng.choice([4, 8]))
    bits = int(rng.choice([8, 12, 16]))
    R = int(rng.choice([1, 2, 3, 4]))
    E = int(rng.choice([16, 100, 256])) if bits == 8 else int(rng.choice([256, 1000, 4096]))
    tile = None
    if bits != 12 and rng.random() < 0.3:
        tile = (int(rng.choice([16, 32, 64])), int(rng.choice([64, 128])))
    if (bits == 12 or tile) and R == 3:
        R = 2                                   # those formats take 1, 2 or 4 codebooks
    if bits == 12 and R * E * v * 2 > 128 * 1024:
        E = 1000                                # 12-bit codes: all codebooks in LDS
    kmul = tile[1] if tile else 8 * v
    K = int(rng.integers(1, 9)) * kmul
    if bits == 12:
        while ((K // v) * R) % 8:
            K += kmul
    if tile and (K // tile[1]) * R * E * v * 2 > 128 * 1024:
        E = 64
    N = int(rng.integers(1, 200))
    return N, K, v, bits, R, E, tile


@pytest.mark.parametrize("N,K,v,bits,R,E,tile,bs", [
    (8200, 512, 8, 8, 2, 256, None, 16),        # 257 workgroups of 32 rows, the last one with 8 rows
    (8192, 1024, 4, 8, 1, 256, None, 11),       # v = 4, batch not a power of two
    (8192, 512, 8, 12, 2, 4096, None, 16),      # packed 12-bit codes, two 64 KiB codebooks
    (9000, 256, 8, 16, 1, 4096, None, 8),       # uint16 codes, one codebook in LDS
    (8208, 512, 8, 8, 4, 256, None, 9),         # four codebooks; 8208 = 256.5 * 32: a workgroup with one tile
    (8192, 512, 4, 8, 1, 256, (256, 256), 16),  # one codebook per (256, 256) tile
    (11008, 4096, 8, 8, 2, 256, None, 16),      # the Llama-7B gate/up shape of the additive configuration
])
def test_gemv_batched_two_row_tiles_per_workgroup(gpu_device, N, K, v, bits, R, E, tile, bs):
    # many rows and a batch: a workgroup takes two 16-row tiles that share their x operands
    w = wl.make_weight(N, K, v, bits, R, E, 0.02, seed=9500 + N + bs, cb_tile=tile)
    wd = vq.weight_to_device(w, gpu_device)
    x = wl.make_activations(bs, K, 9501 + bs)
    want = oracle.gemv(ocodes(w), w.codebooks, w.scale, x, cb_tile=tile)
    got = vq.vq_gemv(wd, dev_x(x, gpu_device))
    torch.cuda.synchronize()
    assert_close(got, want, f"N{N} K{K} v{v} bits{bits} R{R} E{E} tile{tile} bs{bs}")
    # the same rows one token at a time (one tile per workgroup): same sums up to the order of the wavefronts' parts
    one = vq.vq_gemv(wd, dev_x(x[:1].copy(), gpu_device))
    torch.cuda.synchronize()
    assert_close(one, want[:1], "first token alone")


@pytest.mark.parametrize("seed", range(int(__import__("os").environ.get("VQ_TEST_RANDOM_CASES", "24"))))
def test_gemv_gemm_dequant_random_formats(gpu_device, seed):
    rng = np.random.default_rng(97000 + seed)
    N, K, v, bits, R, E, tile = _random_weight_case(rng)
    w = wl.make_weight(N, K, v, bits, R, E, 0.02, seed=97100 + seed, with_scale=bool(rng.random() < 0.7), cb_tile=tile)
    what = f"N{N} K{K} v{v} bits{bits} R{R} E{E} tile{tile}"
    wd = vq.weight_to_device(w, gpu_device)
    want32 = oracle.dequant(ocodes(w), w.codebooks, cb_tile=tile)
    got32 = vq.vq_dequant(wd, out_fp32=True)
    torch.cuda.synchronize()
    assert got32.cpu().numpy().tobytes() == want32.tobytes(), what
    for bs in (1, int(rng.integers(2, 17))):
        x = wl.make_activations(bs, K, 97200 + seed + bs)
        assert_close(vq.vq_gemv(wd, dev_x(x, gpu_device)),
                     oracle.gemv(ocodes(w), w.codebooks, w.scale, x, cb_tile=tile), what + f" bs{bs}")
    M = int(rng.choice([20, 70, 270]))
    X = wl.make_activations(M, K, 97300 + seed)
    assert_close(vq.vq_gemm(wd, dev_x(X, gpu_device)),
                 oracle.gemm(ocodes(w), w.codebooks, w.scale, X, cb_tile=tile), what + f" M{M}")


@pytest.mark.parametrize("seed", range(int(__import__("os").environ.get("VQ_TEST_RANDOM_CASES", "16"))))
def test_attn_random_shapes(gpu_device, seed):
    rng = np.random.default_rng(98000 + seed)
    v = int(rng.choice([2, 4, 8]))
    P = 128 // v
    G = int(rng.choice([g for g in (1, 2, 4, 8, 16, 32, 64) if P % g == 0 and g * 256 * v * 2 <= 64 * 1024]))
    B, H = int(rng.integers(1, 6)), int(rng.integers(1, 5))
    T = int(rng.choice([1, 17, 255, 256, 257, 1000, 1536, 3000]))
    E = int(rng.choice([16, 200, 256]))
    kv = wl.make_kv(B, H, 128, T, v, E, G, seed=98100 + seed, ragged=bool(rng.random() < 0.5))
    if kv.seq_lens is not None and rng.random() < 0.3:
        kv.seq_lens[int(rng.integers(0, B))] = 0
    sm = float(rng.choice([1.0 / np.sqrt(128.0), 0.3]))
    assert_close(run_attn(kv, gpu_device, sm), oracle_attn(kv, sm), f"attn B{B} H{H} T{T} v{v} G{G} E{E}")


@pytest.mark.parametrize("seed", range(int(__import__("os").environ.get("VQ_TEST_RANDOM_CASES", "12"))))
def test_gemv_packed_random_shapes(gpu_device, seed):
    rng = np.random.default_rng(99000 + seed)
    E = int(rng.choice([4096, 8192, 16384, 65536]))
    K = int(rng.integers(1, 40)) * 64 if rng.random() < 0.7 else int(rng.integers(1, 255)) * 8 * 8
    K = min(K, 2047 * 8)
    N = int(rng.choice([1, 63, 64, 65, 500, 1500, 4097]))
    zipf = float(rng.choice([0.8, 1.2])) if rng.random() < 0.3 else None
    count = int(rng.integers(1, 5))
    ws = [wl.make_weight(N if i == 0 else int(rng.integers(1, 700)), K, 8, 16, 1, E, 0.02, seed=99100 + 10 * seed + i,
                         with_scale=bool(rng.random() < 0.7), zipf_s=zipf) for i in range(count)]
    x = wl.make_activations(1, K, 99200 + seed)
    xd = dev_x(x, gpu_device)
    # (skewed codes may be declined by the re-tiling: those members run from their canonical codes)
    packable = [vq.vq_gemv_prepack(w)[0] is not None for w in ws]
    assert zipf is not None or all(packable)
    wds = [vq.weight_to_device(w, gpu_device, prepack=ok, keep_codes=not ok) for w, ok in zip(ws, packable)]
    ys = vq.vq_gemv_batch(wds, [xd] * count)
    torch.cuda.synchronize()
    for i, (w, wd, y) in enumerate(zip(ws, wds, ys)):
        what = f"packed N{w.N} K{K} E{E} zipf{zipf} member {i}/{count} packed={packable[i]}"
        assert_close(y, oracle.gemv(w.codes, w.codebooks, w.scale, x), what)
        assert torch.equal(y, vq.vq_gemv(wd, xd)), what


@pytest.mark.parametrize("seed", range(int(__import__("os").environ.get("VQ_TEST_RANDOM_CASES", "16"))))
def test_kv_quantize_random_shapes(gpu_device, seed):
    rng = np.random.default_rng(96000 + seed)
    v = int(rng.choice([2, 4, 8]))
    P = 128 // v
    G = int(rng.choice([g for g in (1, 2, 4, 8, 16, 32, 64) if P % g == 0 and g * 256 * v * 2 <= 64 * 1024]))
    E = int(rng.choice([8, 16, 200, 256]))
    if (G * E * v * 2) % 16 != 0:
        E = 256
    B, H = int(rng.integers(1, 5)), int(rng.integers(1, 5))
    n_new = int(rng.choice([1, 1, 2, 3, 7, 8, 9, 64, 65, 150]))
    T = n_new + int(rng.integers(0, 40))
    pos = int(rng.integers(0, T - n_new + 1))
    kv = wl.make_kv(B, H, 128, T, v, E, G, seed=96100 + seed)
    if rng.random() < 0.3:      # some repeated entries: exact ties
        for cb in (kv.k_codebooks, kv.v_codebooks):
            cb[:, :, E // 2:, :] = cb[:, :, :E - E // 2, :]
    k_new = rng.normal(0, 1, size=(B, H, n_new, 128)).astype(np.float16)
    v_new = rng.normal(0, 1, size=(B, H, n_new, 128)).astype(np.float16)
    what = f"kvq B{B} H{H} T{T} v{v} G{G} E{E} n_new{n_new} pos{pos}"
    kd = vq.kv_to_device(kv, gpu_device)
    vq.vq_kv_quantize(kd, dev_x(k_new, gpu_device), dev_x(v_new, gpu_device), pos)
    torch.cuda.synchronize()
    want_k, want_v = kv.k_codes.copy(), kv.v_codes.copy()
    want_k[:, :, pos:pos + n_new] = oracle.kv_quantize(k_new, kv.k_codebooks)
    want_v[:, :, pos:pos + n_new] = oracle.kv_quantize(v_new, kv.v_codebooks)
    assert np.array_equal(kd.k_codes.cpu().numpy(), want_k), what
    assert np.array_equal(kd.v_codes.cpu().numpy(), want_v), what


# ---------------------------------------------------------------- measurement probes

def test_measurement_probes_run_and_copy_is_exact(gpu_device):
    # vq_probe_copy is what the HBM counters are calibrated on: it must move exactly the bytes it is given
    src = torch.randint(0, 256, (1 << 20,), dtype=torch.uint8, device=gpu_device)
    dst = torch.zeros_like(src)
    vq.vq_probe_copy(dst, src)
    sink = torch.zeros(1 << 16, dtype=torch.uint8, device=gpu_device)
    vq.vq_probe_read(src, sink)
    for mode in (0, 1, 2):      # smooth register operands, random register operands, random operands from LDS
        vq.vq_probe_mfma(8, 4, sink, random_operands=mode)
    torch.cuda.synchronize()
    assert torch.equal(dst, src)


def test_gemv_pipeline_small_codebook_list_as_replayed_graph(gpu_device):
    """The small-codebook kind of vq_gemv_pipeline captured into a HIP graph and replayed, with eager work and
    synchronisations in between: every replay gives the bits of the eager run."""
    calls, ref = [], []
    for i, (N, K) in enumerate([(4096, 1024), (1000, 2112), (2500, 512), (300, 11008), (4096, 4096)]):
        w = wl.make_weight(N, K, 8, 8, 2, 256, 0.01, seed=9700 + i)
        xd = dev_x(wl.make_activations(1, K, seed=9750 + i), gpu_device)
        calls.append([(vq.weight_to_device(w, gpu_device), xd, torch.full((1, N), 7.0, dtype=torch.float16, device=gpu_device))])
        ref.append((w, xd))
    pipe = vq.GemvPipeline(calls)
    assert pipe.run() == 0
    torch.cuda.synchronize()
    want = [c[0][2].clone() for c in calls]
    for c, (w, xd) in zip(calls, ref):
        assert_close(c[0][2], oracle.gemv(w.codes, w.codebooks, w.scale, xd.cpu().numpy()), f"eager {w.N}x{w.K}")
        c[0][2].fill_(7.0)
    g = torch.cuda.CUDAGraph()
    cap = torch.cuda.Stream()
    with torch.cuda.stream(cap):
        with torch.cuda.graph(g, stream=cap):
            assert pipe.run() == 0
    for rep in range(4):
        g.replay()
        torch.cuda.synchronize()
        for c, w_ in zip(calls, want):
            assert torch.equal(c[0][2], w_), rep
            c[0][2].fill_(7.0)
        vq.vq_gemv(calls[0][0][0], calls[0][0][1])           # eager work of the program between the replays
        torch.cuda.synchronize()
    del g
    pipe.close()


# Long ranges with copies of the codebooks: weights without a running maximum where the scores are bounded, with one where they are
# not (a large scale, or an entry that is infinite, used or not); empty, one-token and ragged sequences
@pytest.mark.parametrize("kind", ["bounded", "near_the_bound", "large_scale", "infinite_entry_unused", "nan_entry_unused", "negative_scale"])
def test_attn_decode_bounded_scores(gpu_device, kind):
    B, H, T, D, v, E = 16, 32, 4096, 128, 4, 256
    from paper_2503_02236_amd.binding import vq_kv_t
    g = torch.Generator(device=gpu_device).manual_seed(8800)
    codes = [torch.randint(0, E - 1, (B, H, T, D // v), generator=g, device=gpu_device, dtype=torch.int32).to(torch.uint8) for _ in range(2)]
    cb = [torch.randn((H, 1, E, v), generator=g, device=gpu_device).to(torch.float16) for _ in range(2)]
    q = torch.randn((B, H, D), generator=g, device=gpu_device).to(torch.float16)
    scale = {"near_the_bound": 0.16, "large_scale": 2.5, "negative_scale": -0.09}.get(kind, 0.088)
    if "unused" in kind:    # (no code is E - 1)
        cb[0][:, 0, E - 1, 1] = float("inf") if kind.startswith("inf") else float("nan")
        cb[1][:, 0, E - 1, 0] = float("nan")
    kv = vq.VQKVDev(B, H, D, T, v, codes[0], codes[1], cb[0], cb[1])
    kv.seq_lens = torch.tensor([0, 1, 33, 4095] + [4096 - 300 * i for i in range(12)], dtype=torch.int32, device=gpu_device)
    import ctypes as ct
    d = kv.desc()
    f = vq.lib()._ZN2vq15attn_replicatedEPK7vq_kv_t
    f.restype = ct.c_bool
    assert f(ct.byref(d)) and isinstance(d, vq_kv_t)
    out = vq.vq_attn_decode(kv, q, scale).double().cpu()
    assert (out[0] == 0).all()
    for b, h in [(1, 0), (2, 31), (3, 7), (4, 0), (9, 16), (15, 31)]:
        n = int(kv.seq_lens[b])
        K, V = (cb[i][h, 0].double().cpu()[codes[i][b, h, :n].long().cpu()].reshape(n, D) for i in range(2))
        p = torch.softmax(scale * (K @ q[b, h].double().cpu()), 0)
        assert_close(out[b, h], (p @ V).numpy(), f"{kind} b{b} h{h}")


# ---------------------------------------------------------------- native marshalling of the Python calls

def _both_ways(monkeypatch, f):
    """f() as it is and with ctypes alone: (result or exception) of each."""
    from paper_2503_02236_amd import binding
    vq.lib()
    assert binding._marshal is not None, "the native part of the binding is not built"
    got = []
    for native in (binding._marshal, None):
        monkeypatch.setattr(binding, "_marshal", native)
        try:
            r = f()
            torch.cuda.synchronize()
        except Exception as e:  # noqa: BLE001
            r = (type(e), str(e))
        got.append(r)
    monkeypatch.undo()
    return got


def _same(a, b):
    if isinstance(a, (list, tuple)):
        return type(a) is type(b) and len(a) == len(b) and all(_same(x, y) for x, y in zip(a, b))
    if isinstance(a, torch.Tensor):
        return a.dtype == b.dtype and a.shape == b.shape and a.stride() == b.stride() and a.device == b.device and torch.equal(a, b)
    return a == b


@pytest.mark.parametrize("fmt", ["u8x2", "u12x2", "u16", "pack", "tile"])
def test_native_marshalling_gemv_gemm(gpu_device, monkeypatch, fmt):
    v, bits, R, E = {"u8x2": (8, 8, 2, 256), "u12x2": (8, 12, 2, 4096), "u16": (8, 16, 1, 65536), "pack": (8, 16, 1, 65536), "tile": (4, 8, 1, 256)}[fmt]
    if fmt == "tile":
        wd = vq.weight_to_device(wl.gptvq_like_layer(0), gpu_device)
    else:
        w = wl.make_weight(512, 1024, v, bits, R, E, 0.02, seed=77, with_scale=fmt != "u16")
        wd = vq.weight_to_device(w, gpu_device, prepack=fmt == "pack")
    K = wd.K
    x1, x5, X = (dev_x(wl.make_activations(n, K, seed=78 + n), gpu_device) for n in (1, 5, 300))
    for f in (lambda: vq.vq_gemv(wd, x1), lambda: vq.vq_gemv(wd, x5), lambda: vq.vq_gemm(wd, X), lambda: vq.vq_gemm(wd, X=X[:40].contiguous()),
              lambda: vq.vq_gemv_batch([wd, wd], [x1, x1]), lambda: vq.vq_gemv_batch((wd, wd), (x1, x1)),
              # refused, or taken, alike: shapes, types, strides, scratch, host memory
              lambda: vq.vq_gemv(wd, X), lambda: vq.vq_gemv(wd, x1.float()), lambda: vq.vq_gemv(wd, x5.t()), lambda: vq.vq_gemv(wd, x1.cpu()),
              lambda: vq.vq_gemm(wd, X, ws=torch.empty(16, dtype=torch.uint8, device=gpu_device)), lambda: vq.vq_gemv(wd, x5[:0]),
              lambda: vq.vq_gemv(wd, x1, y=torch.empty((1, wd.N), device=gpu_device)), lambda: vq.vq_gemv_batch([wd], [x1, x1]),
              lambda: vq.vq_gemv_batch([], []), lambda: vq.vq_gemv(wd, x5[:, 1:]), lambda: vq.vq_gemv(wd, None)):
        a, b = _both_ways(monkeypatch, f)
        assert _same(a, b), (fmt, a, b)
    y = torch.empty((5, wd.N), dtype=torch.float16, device=gpu_device)
    assert vq.vq_gemv(wd, x5, y=y) is y and vq.vq_gemm(wd, X[:5].contiguous(), Y=y) is y
    ys = [torch.empty((1, wd.N), dtype=torch.float16, device=gpu_device) for _ in range(2)]
    assert vq.vq_gemv_batch([wd, wd], [x1, x1], ys) is ys
    s = torch.cuda.Stream()
    want = vq.vq_gemv(wd, x5)
    torch.cuda.synchronize()
    with torch.cuda.stream(s):
        got = vq.vq_gemv(wd, x5)
    s.synchronize()
    assert torch.equal(got, want)


def test_native_marshalling_attention(gpu_device, monkeypatch):
    kv, q = wl.make_kv(2, 3, 128, 204, 4, 256, 1, seed=91), dev_x(wl.make_activations(6, 128, seed=92), gpu_device).view(2, 3, 128)
    kd = vq.kv_to_device(kv, gpu_device)
    new = torch.randn((2, 3, 4, 128), device=gpu_device).to(torch.float16)

    def quantize(*args):
        vq.vq_kv_quantize(kd, *args)
        return kd.k_codes.clone(), kd.v_codes.clone()
    for f in (lambda: vq.vq_attn_decode(kd, q, 0.09), lambda: vq.vq_attn_decode(kd, q, 1), lambda: vq.vq_attn_decode(kd, q.float(), 0.09),
              lambda: vq.vq_attn_decode(kd, q.transpose(0, 1), 0.09), lambda: quantize(new, new * 0.5, 7), lambda: quantize(new, new, 199),
              lambda: quantize(new, new.float(), 0), lambda: quantize(new, new, 3.0), lambda: quantize(new[:, :, :0], new, 0)):
        a, b = _both_ways(monkeypatch, f)
        assert _same(a, b), (a, b)
    kd.seq_lens = torch.tensor([150, 3], dtype=torch.int32, device=gpu_device)
    a, b = _both_ways(monkeypatch, lambda: vq.vq_attn_decode(kd, q, 0.09))
    assert _same(a, b)
    kd.seq_lens = torch.tensor([150, 3], device=gpu_device)      # int64: refused
    a, b = _both_ways(monkeypatch, lambda: vq.vq_attn_decode(kd, q, 0.09))
    assert a == b and a[0] is TypeError


def test_native_marshalling_holds_what_the_lists_of_a_batch_held(gpu_device):
    """The interpreter's lock is released around the entry point, so another thread may change the caller's lists meanwhile: here the
    entry point is a stand-in that does so, and all weights, inputs and outputs have to be there still."""
    import weakref
    from paper_2503_02236_amd import binding
    l, native = vq.lib(), binding._marshal
    names = ("vq_gemv", "vq_gemv_workspace", "vq_gemv_batch", "vq_gemv_batch_workspace", "vq_gemm", "vq_gemm_workspace", "vq_attn_decode",
             "vq_attn_decode_workspace", "vq_kv_quantize")
    address = [ctypes.cast(getattr(l, n), ctypes.c_void_p).value for n in names]
    types = (vq.VQWeightDev, vq.VQKVDev, binding.vq_gemv_pack_t, vq.VQError)
    w, _ = wl.config1_tiny()
    ws = [vq.weight_to_device(w, gpu_device) for _ in range(3)]
    xs = [torch.zeros((1, w.K), dtype=torch.float16, device=gpu_device) for _ in range(3)]
    ys = [torch.zeros((1, w.N), dtype=torch.float16, device=gpu_device) for _ in range(3)]
    refs, alive = [weakref.ref(o) for o in ws + xs + ys], []

    def entry(*args):
        ws.clear(), xs.clear(), ys.clear()
        alive.append(all(r() is not None for r in refs))
        return 0
    stand_in = ctypes.CFUNCTYPE(ctypes.c_int, *l.vq_gemv_batch.argtypes)(entry)
    try:
        native.init(tuple(address[:2] + [ctypes.cast(stand_in, ctypes.c_void_p).value] + address[3:]), *types)
        assert native.gemv_batch(ws, xs, ys, None) is ys
    finally:
        native.init(tuple(address), *types)
    assert alive == [True] and not any(r() for r in refs)


def test_native_marshalling_leaves_what_is_not_plain_to_python(gpu_device):
    from paper_2503_02236_amd import binding
    from torch.overrides import TorchFunctionMode
    w, x = wl.config1_tiny()
    wd, x = vq.weight_to_device(w, gpu_device), dev_x(x, gpu_device)
    native = binding._marshal

    class Sub(torch.Tensor):
        pass

    class SubWeight(vq.VQWeightDev):
        pass

    class Mode(TorchFunctionMode):
        seen = 0

        def __torch_function__(self, func, types, args=(), kwargs=None):
            Mode.seen += "new_empty" in str(func)
            return func(*args, **(kwargs or {}))
    want = vq.vq_gemv(wd, x)
    sub = SubWeight(**{f: getattr(wd, f) for f in wd.__dataclass_fields__})
    assert native.gemv(wd, x, None, None) is not NotImplemented
    assert native.gemv(wd, x.as_subclass(Sub), None, None) is NotImplemented and native.gemv(sub, x, None, None) is NotImplemented
    assert torch.equal(vq.vq_gemv(sub, x), want)
    with Mode():
        assert native.gemv(wd, x, None, None) is NotImplemented
        assert torch.equal(vq.vq_gemv(wd, x), want)
    assert Mode.seen == 1
    g = torch.cuda.CUDAGraph()          # captured like any other call
    y = torch.zeros_like(want)
    vq.vq_gemv(wd, x, y=y)
    with torch.cuda.graph(g):
        vq.vq_gemv(wd, x, y=y)
    for _ in range(3):
        y.zero_()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, want)
