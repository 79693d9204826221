"""Parity of the HIP path with the CPU oracle, element by element, through the C ABI.

Bar: packed codes, headers, group statistics and bit allocations bit-exact; dequantized
values bit-exact as well (both sides evaluate one fused multiply-add in binary32 and one
round-to-nearest conversion to binary16), which is inside the stated 1e-6 / 1e-3 relative
tolerance; the tolerance itself is also asserted so a later relaxation stays bounded.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2104_14129_amd import binding as B
from paper_2104_14129_amd import synth
from _gpu import GpuRun

pytestmark = pytest.mark.gpu


def _assert_dequant(got, want, header, bits, tol):
    """Bit equality expected; and in any case within `tol` of the group magnitude."""
    N, D = want.shape
    ng = header.shape[1]
    Bn = (2.0 ** bits.astype(np.float64) - 1)[:, None]
    mag = np.maximum(np.abs(header[:, :, 0]), np.abs(header[:, :, 0] + Bn * header[:, :, 1])).astype(np.float64)
    mag = np.repeat(mag, 256, axis=1)[:, :D]
    err = np.abs(got.astype(np.float64) - want.astype(np.float64))
    assert np.all(err <= tol * np.maximum(mag, np.finfo(np.float32).tiny))
    assert np.array_equal(got.view(np.uint8), want.view(np.uint8))


def _round_trip(x, bits, seed, tag, noise_bits, out_dtypes=(torch.float32,)):
    run = GpuRun(x, bits)
    N, D = run.N, run.D
    x2 = x.reshape(N, D)
    # a1
    gmin, grange = run.stats()
    omin, orange = oracle.group_stats(x2)
    assert np.array_equal(gmin.view(np.uint32), omin.view(np.uint32))
    assert np.array_equal(grange.view(np.uint32), orange.view(np.uint32))
    # a2-a5
    packed, header = run.quantize(seed, tag, noise_bits)
    opacked, oheader, ooff = oracle.quantize_pack(x2, bits, seed, tag, noise_bits=noise_bits)
    assert np.array_equal(run.offsets_np, ooff) and run.total == opacked.size
    assert np.array_equal(header.view(np.uint32), oheader.view(np.uint32))
    if not np.array_equal(packed, opacked):
        bad = np.flatnonzero(packed != opacked)
        raise AssertionError(f"{bad.size} packed bytes differ, first at {bad[:8]}")
    # a6-a7
    for dt in out_dtypes:
        npdt = np.float32 if dt == torch.float32 else np.float16
        out = run.dequantize(dt)
        want = oracle.unpack_dequantize(opacked, oheader, bits, ooff, N, D, out_dtype=npdt)
        _assert_dequant(out, want, oheader, bits, 1e-6 if dt == torch.float32 else 1e-3)
    return run


def test_smoke_library_is_the_hip_one():
    assert B.version() >= 200
    assert torch.cuda.is_available()


@pytest.mark.parametrize("noise_bits", [24, 16])
def test_config1_tiny(noise_bits):
    wl = synth.tiny()
    x = synth.make_input(wl)
    _round_trip(x, wl.bits, wl.philox_seed, wl.tag, noise_bits, (torch.float32, torch.float16))


@pytest.mark.parametrize("dtype", [np.float32, np.float16])
@pytest.mark.parametrize("noise_bits", [24, 16])
@pytest.mark.parametrize("N,D", [(5, 256 * 7), (3, 256 * 13 + 100), (2, 257), (4, 255), (1, 4 * 256 + 1),
                                 (7, 256 * 33 + 252), (9, 256),
                                 # whole groups around the eight groups a wavefront takes for binary16 output
                                 (2, 256 * 8), (2, 256 * 9), (3, 256 * 15), (2, 256 * 16), (2, 256 * 17), (4, 256 * 3)])
def test_shapes_spanning_tiles_and_ragged_tails(N, D, noise_bits, dtype):
    rng = np.random.default_rng(N * 1000 + D)
    x = (rng.standard_normal((N, D)) * np.exp(rng.uniform(-3, 3, (N, 1)))).astype(dtype)
    bits = rng.integers(1, 9, N).astype(np.uint8)
    _round_trip(x, bits, seed=0xDEADBEEFCAFE + D, tag=(7 << 32) | N, noise_bits=noise_bits,
                out_dtypes=(torch.float32, torch.float16))


@pytest.mark.parametrize("b", [1, 2, 3, 4, 5, 6, 7, 8])
def test_each_width_uniform_many_tiles(b):
    rng = np.random.default_rng(b)
    N, D = 6, 256 * 70
    x = np.maximum(rng.standard_normal((N, D)), 0).astype(np.float32)
    _round_trip(x, np.full(N, b, dtype=np.uint8), seed=b, tag=b, noise_bits=24)
    _round_trip(x, np.full(N, b, dtype=np.uint8), seed=b, tag=b, noise_bits=16)


def test_degenerate_groups_negative_zero_and_subnormals():
    N, D = 4, 256 * 6
    rng = np.random.default_rng(11)
    x = rng.standard_normal((N, D)).astype(np.float32)
    x[0, :256] = 3.25                                   # constant group
    x[0, 256:512] = 0.0
    x[0, 300] = -0.0                                    # min is -0.0
    x[3, 512:768] = 0.0
    x[3, 512:768:2] = -0.0                              # zeros of both signs, -0.0 first: range is +0.0
    x[1, :256] = np.float32(1e-45) * rng.integers(0, 2, 256)      # range = smallest subnormal
    x[1, 256:512] = (rng.integers(0, 1000, 256) * np.float32(1e-42)).astype(np.float32)  # subnormal data
    x[2, :256] = -np.abs(x[2, :256])
    x[2, 10] = -0.0                                     # max is -0.0
    x[3, :512] = np.float32(1e30) * rng.standard_normal(512).astype(np.float32)
    for b in (1, 2, 3, 4, 7, 8):
        run = _round_trip(x, np.full(N, b, dtype=np.uint8), seed=5, tag=0, noise_bits=24)
        hd = run.header.cpu().numpy().reshape(N, -1, 2)
        assert hd[0, 0, 1] == 0.0 and hd[0, 1, 0] == 0.0 and not np.signbit(hd[0, 1, 0])
        assert hd[1, 0, 1] == 0.0       # B / R overflowed: degenerate


def test_degenerate_groups_binary16_with_16_bit_noise():
    """The binary16 kernel's own corner cases: constant groups, zeros of both signs, subnormal data,
    the largest finite values of both signs in one group (range 131008 in binary32), a last run of
    fewer than eight groups."""
    N, D = 5, 256 * 11
    rng = np.random.default_rng(12)
    x = rng.standard_normal((N, D)).astype(np.float16)
    x[0, :256] = np.float16(3.25)                        # constant group
    x[0, 256:512] = 0.0
    x[0, 300] = -0.0                                     # min is -0.0
    x[3, 512:768] = 0.0
    x[3, 512:768:2] = -0.0                               # zeros of both signs: range is +0.0
    x[1, :256] = (rng.integers(0, 2, 256) * 6e-8).astype(np.float16)        # range = smallest subnormal
    x[1, 256:512] = (rng.integers(0, 1000, 256) * 6e-8).astype(np.float16)  # subnormal data
    x[2, :256] = -np.abs(x[2, :256])
    x[2, 10] = -0.0                                      # max is -0.0
    x[4, :256] = (rng.uniform(-1, 1, 256) * 65504).astype(np.float16)
    x[4, 0], x[4, 255] = np.float16(65504), np.float16(-65504)
    x[4, 2560:] = np.float16(-7.5)                       # constant group in the short last run
    for b in (1, 2, 3, 4, 5, 6, 7, 8):
        run = _round_trip(x, np.full(N, b, dtype=np.uint8), seed=6, tag=1, noise_bits=16, out_dtypes=(torch.float16,))
        hd = run.header.cpu().numpy().reshape(N, -1, 2)
        assert hd[0, 0, 1] == 0.0 and hd[0, 1, 0] == 0.0 and not np.signbit(hd[0, 1, 0])
        assert hd[4, 10, 0] == -7.5 and hd[4, 10, 1] == 0.0


@pytest.mark.parametrize("case", range(48))
def test_random_full_group_shapes_against_the_oracle(case):
    """Seeded random problems on the kernels that serve full groups: sample counts 1..9, 1..41 groups
    per sample (runs and tiles of every remainder), both input types and noise modes, widths 1..8
    per sample, per-sample scales over six orders of magnitude, some samples constant or all zero."""
    rng = np.random.default_rng(7000 + case)
    N = int(rng.integers(1, 10))
    ng = int(rng.integers(1, 42))
    dtype = np.float16 if case % 2 else np.float32
    noise_bits = 16 if (case // 2) % 2 == 0 else 24
    scale = np.exp(rng.uniform(-7, 7, (N, 1))) if dtype == np.float32 else np.exp(rng.uniform(-5, 5, (N, 1)))
    x = (rng.standard_normal((N, ng * 256)) * scale).astype(dtype)
    if N > 2:
        x[1] = dtype(0.0)
        x[2, :256] = dtype(1.5)
    if case % 3 == 0:
        x = np.maximum(x, dtype(0.0))     # post-ReLU data: many groups with minimum 0
    bits = rng.integers(1, 9, N).astype(np.uint8)
    _round_trip(x, bits, seed=int(rng.integers(0, 2 ** 63)), tag=int(rng.integers(0, 2 ** 40)), noise_bits=noise_bits,
                out_dtypes=(torch.float32, torch.float16))


def test_grid_points_reconstruct_exactly_on_the_gpu():
    N, ng = 4, 8
    rng = np.random.default_rng(3)
    for b in (1, 2, 3, 4, 5, 6, 7, 8):
        Bq = (1 << b) - 1
        k = rng.integers(0, Bq + 1, size=(N, ng, 256))
        k[:, :, 0], k[:, :, 255] = 0, Bq
        x = (-8.0 + k * 0.125).astype(np.float32).reshape(N, ng * 256)
        run = GpuRun(x, np.full(N, b, dtype=np.uint8))
        for seed in (0, 99):
            run.quantize(seed)
            out = run.dequantize()
            assert np.array_equal(out.view(np.uint32), x.view(np.uint32))


def test_samples_with_invalid_width_or_range_are_skipped():
    N, D = 4, 1024
    rng = np.random.default_rng(2)
    x = rng.standard_normal((N, D)).astype(np.float32)
    bits = np.array([2, 2, 2, 2], dtype=np.uint8)
    run = GpuRun(x, bits)
    good_packed, good_header = run.quantize(7)
    # corrupt the DEVICE copies only: width 9 for sample 1, an offset beyond the buffer for sample 2
    run.bits[1] = 9
    run.offsets[2] = run.total - 64
    run.packed_buf.fill_(0xA5)
    run.header_buf.fill_(float("nan"))
    packed, header = run.quantize(7)
    per = run.total // N
    assert np.array_equal(packed[:per], good_packed[:per])
    assert np.all(packed[per:3 * per] == 0xA5)
    assert np.array_equal(packed[3 * per:], good_packed[3 * per:])
    assert np.all(np.isnan(header[1])) and np.all(np.isnan(header[2]))
    assert np.array_equal(header[0], good_header[0]) and np.array_equal(header[3], good_header[3])
    out = run.dequantize()
    assert np.all(np.isnan(out[1])) and np.all(np.isnan(out[2]))
    assert not np.isnan(out[0]).any() and not np.isnan(out[3]).any()


def test_calls_are_reproducible_and_tag_seed_sensitive():
    wl = synth.tiny()
    x = synth.make_input(wl)
    run = GpuRun(x, wl.bits)
    a, _ = run.quantize(1, 0)
    b, _ = run.quantize(1, 0)
    c, _ = run.quantize(2, 0)
    d, _ = run.quantize(1, 1)
    assert np.array_equal(a, b) and not np.array_equal(a, c) and not np.array_equal(a, d)


def test_non_default_stream():
    wl = synth.tiny()
    x = synth.make_input(wl)
    run = GpuRun(x, wl.bits)
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        B.quantize_pack(run.x, run.bits, run.offsets, run.packed, run.header, 1, 0, 24, stream=s)
        out = torch.empty((run.N, run.D), dtype=torch.float32, device="cuda:0")
        B.unpack_dequantize(run.packed, run.header, run.bits, run.offsets, out, stream=s)
    s.synchronize()
    opacked, oheader, ooff = oracle.quantize_pack(x.reshape(run.N, run.D), wl.bits, 1, 0)
    assert np.array_equal(run.packed.cpu().numpy(), opacked)
    want = oracle.unpack_dequantize(opacked, oheader, wl.bits, ooff, run.N, run.D)
    assert np.array_equal(out.cpu().numpy(), want)


# ----------------------------------------------------------------------------- bfloat16 header

def _round_trip_bf16(x, bits, seed, tag, noise_bits, out_dtypes=(torch.float32,)):
    run = GpuRun(x, bits, hf=B.ACTQ_HDR_BF16)
    N, D = run.N, run.D
    x2 = x.reshape(N, D)
    packed, header = run.quantize(seed, tag, noise_bits)
    opacked, oheader, ooff = oracle.quantize_pack_bf16(x2, bits, seed, tag, noise_bits=noise_bits)
    assert np.array_equal(header, oheader)
    assert np.array_equal(packed, opacked)
    for dt in out_dtypes:
        npdt = np.float32 if dt == torch.float32 else np.float16
        out = run.dequantize(dt)
        want = oracle.unpack_dequantize_bf16(opacked, oheader, bits, ooff, N, D, out_dtype=npdt)
        assert np.array_equal(out.view(np.uint8), want.view(np.uint8))
    return run


@pytest.mark.parametrize("dtype", [np.float32, np.float16])
@pytest.mark.parametrize("noise_bits", [24, 16])
@pytest.mark.parametrize("N,D", [(5, 256 * 7), (3, 256 * 13 + 100), (2, 257), (6, 256 * 40), (2, 256 * 9), (3, 256 * 16)])
def test_bf16_header_mode(N, D, noise_bits, dtype):
    rng = np.random.default_rng(N * 77 + D)
    x = (rng.standard_normal((N, D)) * np.exp(rng.uniform(-3, 3, (N, 1))) + rng.standard_normal((N, 1))).astype(dtype)
    bits = rng.integers(1, 9, N).astype(np.uint8)
    _round_trip_bf16(x, bits, seed=11 + D, tag=N, noise_bits=noise_bits, out_dtypes=(torch.float32, torch.float16))


def test_bf16_header_degenerate_groups():
    N, D = 2, 256 * 4
    rng = np.random.default_rng(12)
    x = rng.standard_normal((N, D)).astype(np.float32)
    x[0, :256] = 3.25
    x[0, 256:512] = np.float32(1e-45) * rng.integers(0, 2, 256)
    x[1, :256] = 0.0
    x[1, 7] = -0.0
    for b in (1, 8):
        run = _round_trip_bf16(x, np.full(N, b, dtype=np.uint8), seed=5, tag=0, noise_bits=16)
        hd = run.header.cpu().numpy().reshape(N, -1, 2).view(np.uint16)
        assert hd[0, 0, 1] == 0 and hd[0, 1, 1] == 0 and hd[1, 0, 1] == 0


def test_bf16_header_config2_full_size():
    wl = synth.r50_stage1()
    x = synth.make_input(wl)
    _round_trip_bf16(x.reshape(wl.N, wl.D), wl.bits, wl.philox_seed, wl.tag, 16)


def test_sample_sensitivity_matches_the_oracle():
    """Binary32 sums in a fixed tree order against the oracle's double accumulation: relative
    error of a sum of ng non-negative terms is below (log2(ng) + 8) * 2^-24 < 2e-6."""
    rng = np.random.default_rng(21)
    for N, ng in [(4, 16), (7, 3136), (3, 1), (5, 777)]:
        grange = np.abs(rng.standard_normal((N, ng)) * np.exp(rng.uniform(-4, 4, (N, 1)))).astype(np.float32)
        grad2 = rng.uniform(0.1, 10, N).astype(np.float32)
        g = torch.from_numpy(grange).cuda()
        w = B.sample_sensitivity(g).cpu().numpy()
        assert np.allclose(w, oracle.sample_sensitivity(grange), rtol=2e-6, atol=0)
        w2 = B.sample_sensitivity(g, torch.from_numpy(grad2).cuda()).cpu().numpy()
        assert np.allclose(w2, oracle.sample_sensitivity(grange, grad2=grad2), rtol=2e-6, atol=0)
    # end to end: ranges from group_stats -> sensitivities -> allocator, no host arithmetic in between
    wl = synth.tiny()
    x = torch.from_numpy(synth.make_input(wl).reshape(wl.N, wl.D)).cuda()
    gmin, gr = B.group_stats(x)
    w = B.sample_sensitivity(gr).cpu().numpy()
    bits = B.allocate_bits(w, np.full(wl.N, wl.D, dtype=np.int64), 3 * wl.N * wl.D)
    assert set(bits) <= {1, 2, 4, 8} and int(bits.astype(np.int64).sum()) * wl.D <= 3 * wl.N * wl.D


def test_more_samples_than_one_grid_dimension_holds():
    """N > 65535 exercises the split of the sample index over two grid dimensions."""
    N, D = 70001, 256
    rng = np.random.default_rng(9)
    x = rng.standard_normal((N, D)).astype(np.float32)
    bits = rng.choice([1, 2, 4, 8], N).astype(np.uint8)
    _round_trip(x, bits, seed=3, tag=1, noise_bits=16)
    _round_trip(x[:66000], bits[:66000], seed=3, tag=1, noise_bits=24)


def test_unaligned_device_arrays_are_rejected():
    x = torch.zeros((8, 256), device="cuda:0")
    bits = torch.full((12,), 2, dtype=torch.uint8, device="cuda:0")
    offs = torch.arange(8, dtype=torch.int64, device="cuda:0") * 64
    packed = torch.zeros(8 * 64, dtype=torch.uint8, device="cuda:0")
    header = torch.zeros(8 * 2, device="cuda:0")
    with pytest.raises(B.ActqError) as e:
        B.quantize_pack(x, bits[1:9], offs, packed, header, 1)
    assert e.value.code == B.ACTQ_EINVAL and "bits" in str(e.value)
    with pytest.raises(B.ActqError):
        B.quantize_pack(x.view(-1)[1:257 + 256 * 6].view(7, 256), bits[:7], offs[:7], packed, header[:14], 1)


# ----------------------------------------------------------------------------- per-tensor baseline

@pytest.mark.parametrize("dtype", [np.float32, np.float16])
@pytest.mark.parametrize("n", [1, 3, 4, 7, 255, 4096, 4096 * 33 + 5, 3_000_001])
def test_tensor_stats(n, dtype):
    rng = np.random.default_rng(n)
    x = (rng.standard_normal(n) * 3 + 1).astype(dtype)
    buf = torch.full((4,), float("nan"), dtype=torch.float32, device="cuda:0")
    B.tensor_stats(torch.from_numpy(x).cuda(), buf[:2])
    torch.cuda.synchronize()
    assert torch.isnan(buf[2:]).all()
    assert np.array_equal(buf[:2].cpu().numpy().view(np.uint32), oracle.tensor_stats(x).view(np.uint32))


def test_tensor_stats_negative_zero_and_signs():
    for vals in ([-0.0, 0.0, -0.0, 0.0], [-3.0, -1.0, -2.0, -5.0], [4.0, 2.0, 9.0, 2.5], [-1e-45, 1e-45, 0.0, -0.0]):
        x = np.array(vals * 3, dtype=np.float32)
        zr = B.tensor_stats(torch.from_numpy(x).cuda()).cpu().numpy()
        assert np.array_equal(zr.view(np.uint32), oracle.tensor_stats(x).view(np.uint32)), vals


@pytest.mark.parametrize("dtype", [np.float32, np.float16])
@pytest.mark.parametrize("noise_bits", [24, 16])
@pytest.mark.parametrize("N,D", [(5, 256 * 7), (3, 256 * 13 + 100), (2, 257), (6, 256 * 40)])
def test_per_tensor_mode(N, D, noise_bits, dtype):
    rng = np.random.default_rng(N * 13 + D)
    x = (rng.standard_normal((N, D)) * np.exp(rng.uniform(-3, 3, (N, 1))) + 0.5).astype(dtype)
    bits = rng.integers(1, 9, N).astype(np.uint8)
    run = GpuRun(x, bits, hf=B.ACTQ_HDR_TENSOR)
    zr = oracle.tensor_stats(x)
    B.tensor_stats(run.x, run.header)
    torch.cuda.synchronize()
    assert np.array_equal(run.header.cpu().numpy().view(np.uint32), zr.view(np.uint32))
    packed, header = run.quantize(77, 5, noise_bits)
    assert np.array_equal(header.reshape(-1).view(np.uint32), zr.view(np.uint32)), "the given header must not be written"
    opacked, ooff = oracle.quantize_pack_tensor(x, bits, zr, 77, 5, noise_bits=noise_bits)
    assert np.array_equal(packed, opacked)
    for dt in (torch.float32, torch.float16):
        npdt = np.float32 if dt == torch.float32 else np.float16
        out = run.dequantize(dt)
        want = oracle.unpack_dequantize_tensor(opacked, zr, bits, ooff, N, D, out_dtype=npdt)
        assert np.array_equal(out.view(np.uint8), want.view(np.uint8))


def test_per_tensor_mode_constant_tensor():
    x = np.full((3, 512), -2.5, dtype=np.float32)
    bits = np.array([1, 4, 8], dtype=np.uint8)
    run = GpuRun(x, bits, hf=B.ACTQ_HDR_TENSOR)
    B.tensor_stats(run.x, run.header)
    packed, _ = run.quantize(1)
    assert not packed.any()
    assert np.all(run.dequantize() == -2.5)


def test_variance_sweep_per_group_against_per_tensor():
    """Sec. 4.1's argument measured on the GPU: squared error of one quantization pass per width,
    per-group against per-tensor headers, on group ranges spread over orders of magnitude.  The
    sums over 2^18 elements concentrate, so one pass is compared with the closed-form expectation
    sum scale^2 p (1 - p)."""
    rng = np.random.default_rng(21)
    N, ng, G = 32, 32, 256
    sigma = np.exp(rng.normal(0, 1.5, (N, ng, 1)))
    x = (rng.standard_normal((N, ng, G)) * sigma).astype(np.float32).reshape(N, ng * G)
    gmin, grange = oracle.group_stats(x)
    zr = oracle.tensor_stats(x)
    x64 = x.astype(np.float64)

    def expected(z, scale):
        u = (x64 - z) / np.where(scale > 0, scale, 1.0)
        p = u - np.floor(u)
        return float((scale.astype(np.float64) ** 2 * p * (1 - p)).sum())

    print()
    print("  b   per-group MSE   per-tensor MSE   ratio")
    for b in range(1, 9):
        Bq = np.float32((1 << b) - 1)
        bits = np.full(N, b, dtype=np.uint8)
        pg = GpuRun(x, bits)
        pg.quantize(100 + b, 0, 16)
        se_pg = float(((pg.dequantize().astype(np.float64) - x64) ** 2).sum())
        pt = GpuRun(x, bits, hf=B.ACTQ_HDR_TENSOR)
        B.tensor_stats(pt.x, pt.header)
        pt.quantize(100 + b, 0, 16)
        se_pt = float(((pt.dequantize().astype(np.float64) - x64) ** 2).sum())
        want_pg = expected(np.repeat(gmin, G, axis=1), np.repeat(grange / Bq, G, axis=1))
        want_pt = expected(zr[0], np.full(x.shape, zr[1] / Bq, dtype=np.float32))
        print(f"  {b}   {se_pg / x.size:13.4e}   {se_pt / x.size:14.4e}   {se_pt / se_pg:7.1f}")
        assert abs(se_pg / want_pg - 1) < 0.05 and abs(se_pt / want_pt - 1) < 0.05
        assert se_pt > 10 * se_pg


# ----------------------------------------------------------------------------- samples that end inside a group

# tiles of four groups, runs of eight, the 16-byte pieces (4 or 8 elements) and the lanes' stretches (16, 32) and what
# is left of them; samples aligned to 2, 4, 8, 16, 64 and 128 bytes; one tile, many tiles, several XCD runs
@pytest.mark.parametrize("N,D", [(5, 1), (3, 2), (7, 3), (4, 7), (3, 17), (9, 31), (2, 33), (2, 255), (3, 1023), (3, 1025), (2, 1024 + 16),
                                 (3, 2047), (3, 2049), (2, 2048 + 64), (5, 3 * 1024 + 8), (70, 256 * 33 + 5), (9, 64 * 57 * 57), (40, 3 * 75 * 75)])
@pytest.mark.parametrize("dtype", [np.float32, np.float16])
@pytest.mark.parametrize("noise_bits,hf", [(16, 0), (24, 0), (16, 1), (24, 1), (16, 2), (24, 2)])
def test_ragged_samples_in_every_mode(N, D, dtype, noise_bits, hf):
    rng = np.random.default_rng(N * 31 + D)
    x = (rng.standard_normal((N, D)) * np.exp(rng.uniform(-3, 3, (N, 1))) - 0.25).astype(dtype)
    bits = ((np.arange(N) + D) % 8 + 1).astype(np.uint8)
    if hf == B.ACTQ_HDR_F32:
        _round_trip(x, bits, seed=D, tag=N, noise_bits=noise_bits, out_dtypes=(torch.float32, torch.float16))
    elif hf == B.ACTQ_HDR_BF16:
        _round_trip_bf16(x, bits, seed=D, tag=N, noise_bits=noise_bits, out_dtypes=(torch.float32, torch.float16))
    else:
        run = GpuRun(x, bits, hf=hf)
        zr = oracle.tensor_stats(x)
        run.header.copy_(torch.from_numpy(zr))
        packed, _ = run.quantize(D, N, noise_bits)
        opacked, ooff = oracle.quantize_pack_tensor(x, bits, zr, D, N, noise_bits=noise_bits)
        assert np.array_equal(packed, opacked)
        for dt, npdt in ((torch.float32, np.float32), (torch.float16, np.float16)):
            want = oracle.unpack_dequantize_tensor(opacked, zr, bits, ooff, N, D, out_dtype=npdt)
            assert np.array_equal(run.dequantize(dt).view(np.uint8), want.view(np.uint8))


@pytest.mark.parametrize("ng", [1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 17])
@pytest.mark.parametrize("dtype", [np.float32, np.float16])
@pytest.mark.parametrize("noise_bits,hf", [(16, 0), (24, 1), (16, 2)])
def test_samples_of_few_whole_groups(ng, dtype, noise_bits, hf):
    test_ragged_samples_in_every_mode(41, 256 * ng, dtype, noise_bits, hf)


def _median_us(calls):
    """Each call works on its own tensors, together larger than the Infinity Cache."""
    times = []
    for _ in range(17):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for call in calls:
            call()
        b.record()
        b.synchronize()
        times.append(a.elapsed_time(b) * 1e3 / len(calls))
    return sorted(times[2:])[7]


@pytest.mark.parametrize("hf", [B.ACTQ_HDR_F32, B.ACTQ_HDR_BF16])
def test_dequantizing_samples_of_one_group_takes_little_longer(hf):
    """binary16, 67 MB of mixed widths.  Samples of one group have four times the wavefronts of samples of four: 1.6 times the
    time.  With a run of eight groups of which seven repeat the first, 2.6 times."""
    def us(N, D):
        bits = (1 + torch.arange(N, device="cuda:0") % 8).to(torch.uint8)
        size = bits.long() * (D // 8)
        offsets = torch.cumsum(size, 0) - size
        packed = torch.randint(0, 256, (int(size.sum()),), dtype=torch.uint8, device="cuda:0")
        header = torch.rand(N, D // 256, 2, device="cuda:0")
        if hf == B.ACTQ_HDR_BF16:
            header = header.bfloat16().view(torch.int16)
        sets = [(packed.clone(), header.clone(), torch.empty((N, D), dtype=torch.float16, device="cuda:0")) for _ in range(8)]
        return _median_us([lambda s=s: B.unpack_dequantize(s[0], s[1], bits, offsets, s[2], hf=hf) for s in sets])
    us(131072, 256)
    assert us(131072, 256) < 2.25 * us(32768, 1024)


@pytest.mark.parametrize("N,groups", [(1, 4), (31, 4), (33, 4), (1, 124), (5, 508), (517, 8), (1, 516), (3, 6), (73728, 4), (73729, 4), (145, 2052),
                                      (2049, 148), (1, 294916), (49153, 6)])
def test_statistics_of_whole_tiles_of_binary16(N, groups):
    """Beyond 144 MiB (73728 samples of four groups) their tiles go to the XCDs in runs of their own (of 64 tiles in turn); six groups are not
    whole tiles.  Extremes are exact in binary32."""
    gen = torch.Generator(device="cuda:0").manual_seed(N + groups)
    x = torch.randn(N, 256 * groups, generator=gen, device="cuda:0").half()
    gmin, grange = B.group_stats(x)
    v = x.view(N, groups, 256).float()
    assert torch.equal(gmin.view(N, groups), v.amin(2)) and torch.equal(grange.view(N, groups), v.amax(2) - v.amin(2))


@pytest.mark.parametrize("dtype,groups", [(torch.float32, 3), (torch.float32, 5), (torch.float32, 6), (torch.float32, 9), (torch.float32, 14), (torch.float32, 129),
                                          (torch.float32, 3193), (torch.float16, 5), (torch.float16, 9), (torch.float16, 10), (torch.float16, 28), (torch.float16, 3193)])
@pytest.mark.parametrize("hf", [B.ACTQ_HDR_F32, B.ACTQ_HDR_BF16, B.ACTQ_HDR_TENSOR])
@pytest.mark.parametrize("widths", [(1, 2, 3, 4), (1, 2, 3, 4, 5, 6, 7, 8)])
def test_large_tensors_of_uneven_samples_equal_their_pieces(dtype, groups, hf, widths):
    """Whole groups of which the last tile is short have another order of tiles from 48 MiB on, most of them up to 3.25 bits per element of
    the stream's room; their pieces, and the same stream in a larger room, have that of every tensor."""
    D = 256 * groups
    N = (50 << 20) // (D * torch.finfo(dtype).bits // 8) // 4 * 4
    gen = torch.Generator(device="cuda:0").manual_seed(groups)
    bits = torch.tensor(widths, dtype=torch.uint8, device="cuda:0")[torch.arange(N, device="cuda:0") * 5 % len(widths)]
    size = bits.long() * (D // 8)
    offsets = torch.cumsum(size, 0) - size
    room = torch.randint(0, 256, (N * D,), generator=gen, dtype=torch.uint8, device="cuda:0")
    packed = room[:int(size.sum())]
    tensor = hf == B.ACTQ_HDR_TENSOR
    header = torch.rand(1 if tensor else N, 2 if tensor else groups * 2, generator=gen, device="cuda:0")
    if hf == B.ACTQ_HDR_BF16:
        header = header.bfloat16().view(torch.int16)
    assert N * D * torch.finfo(dtype).bits // 8 >= 48 << 20
    outs = []
    for stream in (packed, room):
        out = torch.full((N * D + 512,), 7.0, dtype=dtype, device="cuda:0")
        B.unpack_dequantize(stream, header.view(-1), bits, offsets, out[:N * D].view(N, D), hf=hf)
        assert (out[N * D:] == 7.0).all()
        outs.append(out)
    out = outs[0]
    assert torch.equal(out.view(torch.uint8), outs[1].view(torch.uint8))
    step = (N + 2) // 3 // 4 * 4
    for n in range(0, N, step):
        part = slice(n, min(N, n + step))
        want = torch.empty((part.stop - n, D), dtype=dtype, device="cuda:0")
        B.unpack_dequantize(packed, (header if tensor else header[part]).reshape(-1), bits[part], offsets[part], want, hf=hf)
        assert torch.equal(out[n * D:part.stop * D].view(-1, D).view(torch.uint8), want.view(torch.uint8)), n


@pytest.mark.parametrize("hf", [B.ACTQ_HDR_F32, B.ACTQ_HDR_BF16])
def test_quantizing_samples_of_three_groups_takes_no_longer(hf):
    """binary32, 134 MB of mixed widths.  A tile holds four groups: with the same number of wavefronts 0.75 of the work and the same
    time as samples of four.  With loads 64 bytes apart in the shorter tile, 1.7 times."""
    def us(N, D):
        bits = (1 + torch.arange(N, device="cuda:0") % 8).to(torch.uint8)
        size = bits.long() * (D // 8)
        offsets = torch.cumsum(size, 0) - size
        sets = [(torch.randn((N, D), device="cuda:0"), torch.empty(int(size.sum()), dtype=torch.uint8, device="cuda:0"),
                 torch.empty(N * (D // 256) * 2, dtype=torch.int16 if hf == B.ACTQ_HDR_BF16 else torch.float32, device="cuda:0"))
                for _ in range(6)]
        return _median_us([lambda s=s: B.quantize_pack(s[0], bits, offsets, s[1], s[2], 1, 2, 16, hf=hf) for s in sets])
    us(43688, 768)
    assert us(43688, 768) < 1.35 * us(32768, 1024)


@pytest.mark.parametrize("dtype", [torch.float32, torch.float16])
def test_more_tiles_than_one_launch_holds(dtype):
    """2^26 + 5 samples of two elements: a tile each, 2^32 lanes, in several launches.  Values 0 and r are grid
    points, so codes, headers and results are known whatever the noise."""
    N = (1 << 26) + 5
    r = 1 + (torch.arange(N, device="cuda:0") % 7).to(dtype)
    x = torch.stack([torch.zeros_like(r), r], dim=1)
    gmin, grange = B.group_stats(x)
    assert not gmin.any() and torch.equal(grange.view(-1), r.float())
    del gmin, grange
    bits = torch.ones(N, dtype=torch.uint8, device="cuda:0")
    offsets = torch.arange(N, device="cuda:0") * 32
    packed = torch.full((N * 32,), 0xA5, dtype=torch.uint8, device="cuda:0")
    header = torch.full((N * 2,), float("nan"), device="cuda:0")
    B.quantize_pack(x, bits, offsets, packed, header, seed=3, noise_bits=16)
    assert (packed.view(N, 32)[:, 0] == 2).all() and not packed.view(N, 32)[:, 1:].any()
    assert not header.view(N, 2)[:, 0].any() and torch.equal(header.view(N, 2)[:, 1], r.float())
    out = torch.full_like(x, float("nan"))
    B.unpack_dequantize(packed, header, bits, offsets, out)
    assert torch.equal(out, x)


@pytest.mark.parametrize("b", [2, 3, 4, 5, 6, 7, 8])
def test_binary16_overshoot_with_the_bfloat16_header(b):
    """A group range that bfloat16 holds exactly and whose scaled maximum lies one ulp above B, on the elements
    with the largest noise: the kernel that clamps for b = 8 only equals the oracle, which always clamps."""
    Bq = np.float32((1 << b) - 1)
    cands = np.arange(0x3800, 0x4000, 8, dtype=np.uint16).view(np.float16)      # eight significant bits
    c32 = cands.astype(np.float32)
    r = cands[np.flatnonzero((c32 * (Bq / c32).astype(np.float32)).astype(np.float32) > Bq)[0]]
    D = 1 << 18
    hits = [d for d in range(D) if oracle.noise(321, 0, 0, d, 16) >= 1.0 - 2.0 ** -16]
    assert hits
    x = np.zeros((1, D), dtype=np.float16)
    x[0, 1::2] = np.float16(float(r) / 2)
    for d in hits:
        x[0, d] = r
        g = d // 256
        if x[0, g * 256:(g + 1) * 256].min() != 0.0:
            x[0, g * 256 + (1 if d % 256 == 0 else 0)] = 0.0
    _round_trip_bf16(x, np.array([b], dtype=np.uint8), 321, 0, 16)


# ----------------------------------------------------------------------------- device allocator

def _oracle_alloc(w, D, budget, widths):
    try:
        return oracle.allocate_bits(w, D, budget, widths), 0
    except oracle.OracleError as e:
        return e.bits, e.code


def _device_alloc(w, D, budget, widths, uniform):
    wd = torch.from_numpy(w).cuda()
    Dd = int(D[0]) if uniform else torch.from_numpy(D).cuda()
    M = w.size
    bits = torch.full((M + 64,), 0xA5, dtype=torch.uint8, device="cuda:0")
    offs = torch.full((M + 8,), -7, dtype=torch.int64, device="cuda:0")
    res = torch.full((2 + 8,), -7, dtype=torch.int64, device="cuda:0")
    B.allocate_bits_device(wd, Dd, budget, widths, bits[:M], offs[:M], res[:2])
    torch.cuda.synchronize()
    assert (bits[M:] == 0xA5).all() and (offs[M:] == -7).all() and (res[2:] == -7).all()
    return bits[:M].cpu().numpy(), offs[:M].cpu().numpy(), int(res[0]), int(res[1])


def _check_alloc(w, D, budget, widths, uniform):
    want, code = _oracle_alloc(w, D, budget, widths)
    got, offs, total, status = _device_alloc(w, D, budget, widths, uniform)
    assert status == code
    if not np.array_equal(got, want):
        bad = np.flatnonzero(got != want)
        raise AssertionError(f"{bad.size} widths differ, first at {bad[:6]}: {got[bad[:6]]} vs {want[bad[:6]]}")
    per = ((D + 255) // 256) * 32 * want.astype(np.int64)
    assert np.array_equal(offs, np.concatenate([[0], np.cumsum(per)[:-1]]))
    assert total == int(per.sum())


@pytest.mark.parametrize("case", range(40))
def test_device_allocator_equals_the_greedy(case):
    rng = np.random.default_rng(5000 + case)
    M = int(rng.choice([1, 2, 7, 64, 128, 500, 1023, 1024, 1025, 3000, 9000, 13000, 20000]))
    w = rng.lognormal(0, 2, M).astype(np.float32)
    if case % 3 == 0:
        w[rng.integers(0, M, M // 3 + 1)] = w[0]                  # equal prices: ties by index
    if case % 4 == 0:
        w[rng.integers(0, M, M // 4 + 1)] = 0.0                   # free items: all their steps tie at 0
    if case % 7 == 0:
        w[:] = np.float32(rng.choice([0.0, 1.0, 1e-38, 1e-45]))   # everything ties, subnormal prices
    uniform = case % 2 == 0
    D = (np.full(M, int(rng.choice([256, 1000, 802816]))) if uniform
         else rng.choice([1, 255, 256, 257, 1024, 25088, 802816], M)).astype(np.int64)
    widths = [B.ACTQ_WIDTHS_POW2, B.ACTQ_WIDTHS_ALL, int(rng.integers(1, 256)) << 1][case % 3]
    lo = min(b for b in range(1, 9) if widths >> b & 1)
    hi = max(b for b in range(1, 9) if widths >> b & 1)
    budget = int(rng.uniform(lo - 0.1, hi + 0.3) * D.sum())
    _check_alloc(w, D, max(budget, 0), widths, uniform)


def _spread(rng, M, law):
    if law == "wide":          # ratios over 60 decades: the bins over w / D are as coarse as they get
        return np.exp(rng.uniform(np.log(1e-30), np.log(1e30), M)).astype(np.float32)
    if law == "close":         # more undecided moves than the kernel lists, all prices different
        return (1.0 + np.arange(M) * 2.0 ** -22).astype(np.float32)
    if law == "groups":        # ninety equal ones each, the groups close together: more than a wavefront of equal prices
        return (1.0 + (np.arange(M) // 90) * 2.0 ** -22).astype(np.float32)
    if law == "few":           # a handful of values: many ties at the threshold, and some free items
        return rng.choice(np.array([0.0, 1e-45, 1.0, 1.0000001, 3.0], dtype=np.float32), M)
    return np.full(M, {"zero": 0.0, "one": 1.0}[law], dtype=np.float32)


# items around the limits of the two kernels: 1024 and 2048 items (one or two per thread of the small kernel, two up to 4096 moves),
# rounds of 4096 items, 16,384 items in registers, one, two and six further rounds; remainders of the quadruples
@pytest.mark.parametrize("law", ["wide", "close", "groups", "few", "zero", "one"])
@pytest.mark.parametrize("M,widths", [(65, 0x102), (128, 0x1FE), (292, 0x1FE), (293, 0x1FE), (682, 0x116), (683, 0x116), (1024, 0x102), (1024, 0x1FE), (1025, 0x102), (1025, 0x1FE), (1337, 0x116),
                                      (1792, 0x11E), (1793, 0x11E), (2047, 0x116), (2048, 0x116), (2049, 0x116), (4096, 0x116),
                                      (4097, 0x1FE), (4099, 0x106), (16384, 0x116), (16385, 0x116), (16390, 0x1FE),
                                      (20480, 0x116), (20481, 0x1FE), (24577, 0x116), (40960, 0x1FE)])
def test_device_allocator_at_the_limits_of_its_kernels(M, widths, law):
    rng = np.random.default_rng(M)
    w = _spread(rng, M, law)
    D = np.full(M, 25088, dtype=np.int64) if law in ("close", "groups") else rng.choice([1, 256, 25088, 802816, 2 ** 34 - 1], M).astype(np.int64)
    lo = min(b for b in range(1, 9) if widths >> b & 1)
    # the host allocator (a heap, checked against the oracle elsewhere) is the reference at these sizes
    for mean in (lo + 0.003, 2.0, 6.7):
        budget = int(mean * float(D.sum()))
        want = B.allocate_bits(w, D, budget, widths)
        got, offs, total, status = _device_alloc(w, D, budget, widths, False)
        assert status == 0 and np.array_equal(got, want), (mean, np.flatnonzero(got != want)[:6])
        per = ((D + 255) // 256) * 32 * want.astype(np.int64)
        assert np.array_equal(offs, np.concatenate([[0], np.cumsum(per)[:-1]])) and total == int(per.sum())


# items on both sides of the number from which on each is tested before it is listed; further rounds with a remainder; lists that hold
# the undecided and lists that overflow
@pytest.mark.parametrize("law", ["log-normal", "wide", "groups", "few"])
@pytest.mark.parametrize("M,widths,uniform", [(131072, 0x1FE, False), (131073, 0x116, False), (131075, 0x1FE, True), (262146, 0x116, True), (400001, 0x1FE, False)])
def test_device_allocator_with_many_items_per_bin(M, widths, uniform, law):
    rng = np.random.default_rng(M)
    w = rng.lognormal(0, 2, M).astype(np.float32) if law == "log-normal" else _spread(rng, M, law)
    D = np.full(M, 25088, dtype=np.int64) if uniform else rng.choice([1, 256, 25088, 802816], M).astype(np.int64)
    for mean in (1.3, 2.0, 6.7):
        budget = int(mean * float(D.sum()))
        want = B.allocate_bits(w, D, budget, widths)
        got, offs, total, status = _device_alloc(w, D, budget, widths, uniform)
        assert status == 0 and np.array_equal(got, want), (mean, np.flatnonzero(got != want)[:6])
        per = ((D + 255) // 256) * 32 * want.astype(np.int64)
        assert np.array_equal(offs, np.concatenate([[0], np.cumsum(per)[:-1]])) and total == int(per.sum())


# sizes of their own beyond 1024 items: two items per thread of the small kernel up to 4096 moves and 2048 items, the large kernel from there
@pytest.mark.parametrize("law", ["wide", "close", "groups", "few", "zero", "one"])
@pytest.mark.parametrize("M,widths", [(1025, 0x11E), (1365, 0x116), (1366, 0x116), (2047, 0x016), (2048, 0x016), (2048, 0x102), (2049, 0x102)])
def test_device_allocator_with_two_items_of_their_own_sizes_per_thread(M, widths, law):
    test_device_allocator_at_the_limits_of_its_kernels(M, widths, law)


# lists of 1 to 64 moves around the threshold, of one price, of several, all different; multiples of four and remainders
@pytest.mark.parametrize("law", ["close", "one", "few", "groups"])
@pytest.mark.parametrize("M", [2, 3, 5, 8, 21, 22, 61, 62, 63, 64, 70])
def test_device_allocator_ranks_lists_of_any_length(M, law):
    w = _spread(np.random.default_rng(M), M, law)
    D = np.full(M, 4096, dtype=np.int64)
    for widths in (0x102, 0x116, 0x1FE):
        for mean in (1.3, 2.0, 3.5, 7.9):
            _check_alloc(w, D, int(mean * M * 4096), widths, True)
            _check_alloc(w, D, int(mean * M * 4096), widths, False)


# items of one size, where the small kernel counts in units of that size: one and two items per thread, the first item beyond
# it, one wavefront and a partial second one; sizes whose reciprocal is exact, is not, and the largest
@pytest.mark.parametrize("law", ["wide", "close", "groups", "few", "zero", "one"])
@pytest.mark.parametrize("M,widths", [(1, 0x1FE), (4, 0x116), (64, 0x1FE), (65, 0x116), (512, 0x102), (1024, 0x1FE), (1025, 0x116),
                                      (2047, 0x1FE), (2048, 0x11E), (2049, 0x1FE)])
def test_device_allocator_of_items_of_one_size(M, widths, law):
    rng = np.random.default_rng(100 + M)
    w = _spread(rng, M, law)
    lo = min(b for b in range(1, 9) if widths >> b & 1)
    for size in (1, 256, 25089, 2 ** 34 - 1):
        D = np.full(M, size, dtype=np.int64)
        for mean in (lo + 0.003, 2.0, 6.7):
            budget = int(mean * M * size)
            want = B.allocate_bits(w, D, max(budget, lo * M * size), widths)   # the host's heap, checked against the oracle elsewhere
            got, offs, total, status = _device_alloc(w, D, max(budget, lo * M * size), widths, True)
            assert status == 0 and np.array_equal(got, want), (size, mean, np.flatnonzero(got != want)[:6])
            per = ((D + 255) // 256) * 32 * want.astype(np.int64)
            assert np.array_equal(offs, np.concatenate([[0], np.cumsum(per)[:-1]])) and total == int(per.sum())


# Runs of neighbours of one size (looked at once per quadruple where a wavefront has nothing else), of lengths that divide a quadruple and not;
# element counts on both sides of where the search (2^29 in units of the sizes' common power of two) and the offsets (2^29 groups) go over to
# 64 bits; an invalid item inside a run.
@pytest.mark.parametrize("law", ["log-normal", "wide", "few"])
@pytest.mark.parametrize("M,run,sizes", [(2049, 4, (256, 25088)), (4097, 7, (256, 25088, 802816)), (13568, 256, (802816, 25088, 100352)), (16384, 300, (512, 1536)),
                                         (4096, 4096, (131071,)), (4096, 4096, (131073,)), (4096, 1024, (2 ** 25, 2 ** 25 - 1)), (4096, 8, (2 ** 25 + 512, 2 ** 25 + 256)),
                                         (16385, 5, (2 ** 23, 2 ** 23 + 1)), (5000, 1, (1, 2 ** 34 - 1))])
def test_device_allocator_of_neighbours_of_one_size(M, run, sizes, law):
    rng = np.random.default_rng(M + run)
    w = rng.lognormal(0, 2, M).astype(np.float32) if law == "log-normal" else _spread(rng, M, law)
    D = np.array([sizes[(i // run) % len(sizes)] for i in range(M)], dtype=np.int64)
    for mean, widths in ((1.2, 0x1FE), (2.0, 0x116), (6.7, 0x1FE)):
        budget = int(mean * float(D.sum()))
        want = B.allocate_bits(w, D, budget, widths)
        got, offs, total, status = _device_alloc(w, D, budget, widths, False)
        assert status == 0 and np.array_equal(got, want), (mean, np.flatnonzero(got != want)[:6])
        per = ((D + 255) // 256) * 32 * want.astype(np.int64)
        assert np.array_equal(offs, np.concatenate([[0], np.cumsum(per)[:-1]])) and total == int(per.sum())
    for bad_w, bad_d in ((np.nan, 0), (-1.0, 0), (1.0, -5), (1.0, 2 ** 34)):
        w2, D2 = w.copy(), D.copy()
        w2[M // 2], D2[M // 2] = bad_w, bad_d or D[M // 2]
        got, offs, total, status = _device_alloc(w2, D2, 2 * int(D.sum()), 0x116, False)
        assert status == B.ACTQ_EINVAL and (got == 1).all()


def test_device_allocator_with_more_than_2_to_the_32_equal_moves():
    """2^30 items of sensitivity 0 with four steps each: 2^32 undecided moves, all at the price of the threshold.  The
    first items go down to one bit until the budget holds, the others keep eight."""
    M = 1 << 30
    w = torch.zeros(M, device="cuda:0")
    bits, offs, res = B.allocate_bits_device(w, 1, 2 * M, 0x11E)
    k, rest = divmod(6 * M, 7)                       # an item frees seven bits; the last one goes 8 -> 4 -> 3 -> 2 -> 1
    assert 0 < rest <= 4 + 1 + 1
    last = 4 if rest <= 4 else (3 if rest <= 5 else 2)
    assert (bits[:k] == 1).all() and int(bits[k]) == last and (bits[k + 1:] == 8).all()
    assert int(res[1]) == 0 and int(res[0]) == 32 * (k + last + 8 * (M - k - 1))
    assert int(offs[0]) == 0 and int(offs[k]) == 32 * k and int(offs[M - 1]) == int(res[0]) - 256


def test_device_allocator_writes_widths_at_any_byte_address():
    M = 5003
    w = synth.lognormal_sensitivities(M, seed=3)
    D = np.full(M, 1000, dtype=np.int64)
    want = B.allocate_bits(w, D, 2 * M * 1000)
    wd = torch.from_numpy(np.concatenate([[0.0], w]).astype(np.float32)).cuda()[1:]    # 4 bytes past an aligned address
    buf = torch.full((M + 9,), 0xA5, dtype=torch.uint8, device="cuda:0")
    bits, offs, res = B.allocate_bits_device(wd, torch.from_numpy(D).cuda(), 2 * M * 1000, bits=buf[1:1 + M])
    assert np.array_equal(bits.cpu().numpy(), want) and int(res[1]) == 0
    assert buf[0] == 0xA5 and (buf[1 + M:] == 0xA5).all()


def test_device_allocator_edges():
    M = 300
    rng = np.random.default_rng(1)
    w = rng.lognormal(0, 2, M).astype(np.float32)
    D = np.full(M, 512, dtype=np.int64)
    P = B.ACTQ_WIDTHS_POW2
    _check_alloc(w, D, 8 * M * 512, P, True)            # exactly loose
    _check_alloc(w, D, 8 * M * 512 - 1, P, True)        # one move
    _check_alloc(w, D, M * 512, P, True)                # exactly everything at one bit
    _check_alloc(w, D, M * 512 - 1, P, True)            # infeasible
    _check_alloc(w, D, 0, P, False)
    _check_alloc(w, D, 3 * M * 512, 1 << 3, True)       # a single allowed width
    _check_alloc(w, D, 3 * M * 512 - 1, 1 << 3, True)
    w[5] = -0.0                                           # negative zero is a valid, free item
    _check_alloc(w, D, 2 * M * 512, B.ACTQ_WIDTHS_ALL, True)
    for bad in (np.nan, np.inf, -1.0):
        w2 = w.copy()
        w2[17] = bad
        got, offs, total, status = _device_alloc(w2, D, 2 * M * 512, P, True)
        assert status == B.ACTQ_EINVAL and np.all(got == 1) and total == M * 2 * 32
    D2 = D.copy()
    D2[3] = 0
    got, offs, total, status = _device_alloc(w, D2, 2 * M * 512, P, False)
    assert status == B.ACTQ_EINVAL and np.all(got == 1)


# more moves than the small kernel takes; the last items lie in the second round beyond the registers
@pytest.mark.parametrize("M", [5003, 20481])
@pytest.mark.parametrize("uniform", [True, False])
def test_large_device_allocator_edges(M, uniform):
    rng = np.random.default_rng(M)
    w = rng.lognormal(0, 2, M).astype(np.float32)
    D = np.full(M, 512, dtype=np.int64)
    P = B.ACTQ_WIDTHS_POW2
    _check_alloc(w, D, 8 * M * 512, P, uniform)            # exactly loose
    _check_alloc(w, D, 8 * M * 512 - 1, P, uniform)        # one move
    _check_alloc(w, D, M * 512, P, uniform)                # exactly everything at one bit
    _check_alloc(w, D, M * 512 - 1, P, uniform)            # infeasible
    _check_alloc(w, D, 0, P, uniform)
    _check_alloc(w, D, 3 * M * 512, 1 << 3, uniform)       # a single allowed width
    _check_alloc(w, D, 3 * M * 512 - 1, 1 << 3, uniform)
    w[[5, M - 2]] = -0.0                                    # negative zero is a valid, free item
    _check_alloc(w, D, 2 * M * 512, B.ACTQ_WIDTHS_ALL, uniform)
    per = np.arange(M) * 64
    for at in (17, M // 2, M - 4098 if M > 16384 else M - 5, M - 1):   # a register round, the first and the second further one
        for bad in (np.nan, np.inf, -1.0):
            w2 = w.copy()
            w2[at] = bad
            got, offs, total, status = _device_alloc(w2, D, 2 * M * 512, P, uniform)
            assert status == B.ACTQ_EINVAL and np.all(got == 1) and np.array_equal(offs, per) and total == M * 64
        if not uniform:
            for size in (0, -7):
                D2 = D.copy()
                D2[at] = size
                got, offs, total, status = _device_alloc(w, D2, 2 * M * 512, P, False)
                assert status == B.ACTQ_EINVAL and np.all(got == 1) and np.array_equal(offs[:at + 1], per[:at + 1])


def test_device_allocator_feeds_the_quantizer_without_a_host_hop():
    """stats -> sensitivity -> device allocator -> quantize -> dequantize on one stream, widths
    and offsets never leaving the device; the result equals the oracle run on the same w."""
    wl = synth.r50_stage1(N=16)
    x_np = synth.make_input(wl).reshape(wl.N, wl.D)
    x = torch.from_numpy(x_np).cuda()
    gmin, gr = B.group_stats(x)
    grad2 = torch.from_numpy(np.random.default_rng(4).lognormal(0, 2, wl.N).astype(np.float32)).cuda()
    w = B.sample_sensitivity(gr, grad2)
    budget = 3 * wl.N * wl.D
    bits, offs, res = B.allocate_bits_device(w, wl.D, budget, B.ACTQ_WIDTHS_ALL)
    ng = (wl.D + 255) // 256
    packed = torch.full((wl.N * ng * 256 + 256,), 0xA5, dtype=torch.uint8, device="cuda:0")   # 8 bits would fit
    header = torch.empty(wl.N * ng * 2, dtype=torch.float32, device="cuda:0")
    out = torch.empty_like(x)
    B.quantize_pack(x, bits, offs, packed[:-256], header, 77, 3, 16)
    B.unpack_dequantize(packed[:-256], header, bits, offs, out)
    torch.cuda.synchronize()
    total, status = int(res[0]), int(res[1])
    assert status == 0 and total * 8 <= budget
    w_np, bits_np = w.cpu().numpy(), bits.cpu().numpy()
    want_bits = oracle.allocate_bits(w_np, np.full(wl.N, wl.D, dtype=np.int64), budget, oracle.WIDTHS_ALL)
    assert np.array_equal(bits_np, want_bits)
    assert len(set(bits_np)) > 2
    opacked, oheader, ooff = oracle.quantize_pack(x_np, want_bits, 77, 3, noise_bits=16)
    assert opacked.size == total and np.array_equal(offs.cpu().numpy().view(np.uint64), ooff)
    assert np.array_equal(packed[:total].cpu().numpy(), opacked)
    assert (packed[total:] == 0xA5).all()
    want = oracle.unpack_dequantize(opacked, oheader, want_bits, ooff, wl.N, wl.D)
    assert np.array_equal(out.cpu().numpy().view(np.uint32), want.view(np.uint32))


def test_device_chain_at_the_benchmark_configuration():
    """The step bench.py times on the stage-1 tensor: group_stats -> sample_sensitivity (with the
    benchmark's gradient norms) -> device allocator; the widths must be the workload's and equal
    the oracle's allocation for the sensitivities the device computed."""
    wl = synth.r50_stage1()
    x = torch.from_numpy(synth.make_input(wl).reshape(wl.N, wl.D)).cuda()
    gmin, grange = B.group_stats(x)
    target = synth.tiered_sensitivities(wl.bits, seed=7)
    unit = B.sample_sensitivity(grange).cpu().numpy().astype(np.float64)
    grad2 = torch.from_numpy((target / unit).astype(np.float32)).cuda()
    w = B.sample_sensitivity(grange, grad2)
    budget = 2 * wl.N * wl.D
    bits, offs, res = B.allocate_bits_device(w, wl.D, budget)
    torch.cuda.synchronize()
    assert int(res[1]) == 0
    assert np.array_equal(bits.cpu().numpy(), wl.bits)
    want = oracle.allocate_bits(w.cpu().numpy(), np.full(wl.N, wl.D, dtype=np.int64), budget)
    assert np.array_equal(bits.cpu().numpy(), want)
    ooff, total = oracle.packed_bytes(wl.N, wl.D, 256, want)
    assert np.array_equal(offs.cpu().numpy().view(np.uint64), ooff) and int(res[0]) == total


def test_device_allocator_full_sweep_size():
    """M = 53 layers x 256 samples with the element counts of the ResNet-50 sweep."""
    shapes = synth.resnet50_conv_input_shapes()
    D = np.repeat(np.array([c * h * w for c, h, w in shapes], dtype=np.int64), 256)
    w = synth.lognormal_sensitivities(D.size, seed=5)
    for widths in (B.ACTQ_WIDTHS_POW2, B.ACTQ_WIDTHS_ALL):
        _check_alloc(w, D, 2 * int(D.sum()), widths, False)


# ----------------------------------------------------------------------------- several tensors per launch

@pytest.mark.parametrize("dtype", [np.float32, np.float16])
@pytest.mark.parametrize("noise_bits,hf", [(16, 0), (24, 0), (16, 1)])
def test_multi_tensor_calls_equal_the_single_tensor_calls(noise_bits, hf, dtype):
    """Five tensors of very different sizes in one launch per kernel: statistics, bit stream,
    headers and dequantized values equal the oracle's (hence the single-tensor calls'), with one
    shared bit stream buffer and tag + i as the tag of tensor i."""
    rng = np.random.default_rng(31 + noise_bits + hf)
    N = 6
    Ds = [256, 256 * 5, 256 * 64, 256 * 3, 256 * 21]
    dev = torch.device("cuda:0")
    tdt = torch.float32 if dtype == np.float32 else torch.float16
    xs_np = [(rng.standard_normal((N, D)) * np.exp(rng.uniform(-2, 2, (N, 1)))).astype(dtype) for D in Ds]
    bits_np = [rng.integers(1, 9, N).astype(np.uint8) for _ in Ds]
    # one bit stream for all tensors: offsets continue from tensor to tensor
    offs_np, base = [], 0
    for D, b in zip(Ds, bits_np):
        o, total = B.packed_bytes(N, D, b)
        offs_np.append(o + np.uint64(base))
        base += total
    packed = torch.full((base + 256,), 0xA5, dtype=torch.uint8, device=dev)
    entries, keep = [], []
    for D, x_np, b, o in zip(Ds, xs_np, bits_np, offs_np):
        ng = D // 256
        e = {"x": torch.from_numpy(x_np).to(dev), "out": torch.full((N, D), float("nan"), dtype=tdt, device=dev),
             "gmin": torch.full((N, ng), float("nan"), dtype=torch.float32, device=dev),
             "grange": torch.full((N, ng), float("nan"), dtype=torch.float32, device=dev),
             "header": (torch.zeros(N * ng * 2, dtype=torch.int16, device=dev) if hf == 1
                        else torch.full((N * ng * 2,), float("nan"), dtype=torch.float32, device=dev)),
             "bits": torch.from_numpy(b).to(dev), "offsets": torch.from_numpy(o.view(np.int64)).to(dev), "D": D}
        entries.append(e)
    table = B.tensor_table(entries)
    code = B.ACTQ_F32 if dtype == np.float32 else B.ACTQ_F16
    B.group_stats_multi(table, code, N)
    B.quantize_pack_multi(table, code, N, packed[:base], seed=77, tag=1000, noise_bits=noise_bits, hf=hf)
    B.unpack_dequantize_multi(table, code, N, packed[:base], hf=hf)
    torch.cuda.synchronize()
    assert (packed[base:] == 0xA5).all()
    pk = packed[:base].cpu().numpy()
    for i, (e, x_np, b, o, D) in enumerate(zip(entries, xs_np, bits_np, offs_np, Ds)):
        omin, orange = oracle.group_stats(x_np)
        assert np.array_equal(e["gmin"].cpu().numpy().view(np.uint32), omin.view(np.uint32)), i
        assert np.array_equal(e["grange"].cpu().numpy().view(np.uint32), orange.view(np.uint32)), i
        if hf == 1:
            opacked, oheader, ooff = oracle.quantize_pack_bf16(x_np, b, 77, 1000 + i, noise_bits=noise_bits)
            want = oracle.unpack_dequantize_bf16(opacked, oheader, b, ooff, N, D, out_dtype=dtype)
            assert np.array_equal(e["header"].cpu().numpy().view(np.uint16), oheader.reshape(-1)), i
        else:
            opacked, oheader, ooff = oracle.quantize_pack(x_np, b, 77, 1000 + i, noise_bits=noise_bits)
            want = oracle.unpack_dequantize(opacked, oheader, b, ooff, N, D, out_dtype=dtype)
            assert np.array_equal(e["header"].cpu().numpy().view(np.uint32), oheader.reshape(-1).view(np.uint32)), i
        lo = int(o[0])
        assert np.array_equal(pk[lo:lo + opacked.size], opacked), i
        assert np.array_equal(e["out"].cpu().numpy().view(np.uint8), want.view(np.uint8)), i


def test_multi_tensor_call_with_the_maximum_number_of_tensors():
    N, D = 3, 512
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(8)
    count = B.MAX_TENSORS_PER_CALL
    xs = [rng.standard_normal((N, D)).astype(np.float32) for _ in range(count)]
    bits = np.full(N, 2, dtype=np.uint8)
    o, total = B.packed_bytes(N, D, bits)
    packed = torch.zeros(total * count, dtype=torch.uint8, device=dev)
    entries = [{"x": torch.from_numpy(x).to(dev), "out": torch.empty((N, D), device=dev),
                "header": torch.empty(N * 2 * 2, device=dev), "bits": torch.from_numpy(bits).to(dev),
                "offsets": torch.from_numpy((o + np.uint64(total * i)).view(np.int64)).to(dev), "D": D}
               for i, x in enumerate(xs)]
    table = B.tensor_table(entries)
    B.quantize_pack_multi(table, B.ACTQ_F32, N, packed, seed=5, tag=0, noise_bits=16)
    B.unpack_dequantize_multi(table, B.ACTQ_F32, N, packed)
    torch.cuda.synchronize()
    pk = packed.cpu().numpy()
    for i in (0, 1, count // 2, count - 2, count - 1):
        opacked, oheader, ooff = oracle.quantize_pack(xs[i], bits, 5, i, noise_bits=16)
        assert np.array_equal(pk[total * i: total * (i + 1)], opacked), i
        want = oracle.unpack_dequantize(opacked, oheader, bits, ooff, N, D)
        assert np.array_equal(entries[i]["out"].cpu().numpy().view(np.uint32), want.view(np.uint32)), i


# ----------------------------------------------------------------------------- under graph capture

def test_the_whole_step_can_be_captured_in_a_graph_and_replayed():
    """The library allocates nothing, never synchronises and clears nothing with memset calls, so a
    caller may capture the step (statistics, sensitivities, device allocator, quantize, dequantize)
    in a HIP graph.  Every replay -- with new data in the same buffers and eager work in between --
    must equal the eager result for that data."""
    wl = synth.r50_stage1(N=16)
    N, D, ng = wl.N, wl.D, wl.ng
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(3)
    x = torch.empty((N, D), dtype=torch.float32, device=dev)
    gmin = torch.empty((N, ng), dtype=torch.float32, device=dev)
    grange = torch.empty((N, ng), dtype=torch.float32, device=dev)
    w = torch.empty(N, dtype=torch.float32, device=dev)
    bits = torch.empty(N, dtype=torch.uint8, device=dev)
    offs = torch.empty(N, dtype=torch.int64, device=dev)
    res = torch.empty(2, dtype=torch.int64, device=dev)
    packed = torch.empty(N * D, dtype=torch.uint8, device=dev)
    header = torch.empty(N * ng * 2, dtype=torch.float32, device=dev)
    out = torch.empty((N, D), dtype=torch.float32, device=dev)
    budget = 3 * N * D

    def step():
        B.group_stats(x, gmin, grange)
        B.sample_sensitivity(grange, None, w)
        B.allocate_bits_device(w, D, budget, B.ACTQ_WIDTHS_ALL, bits, offs, res)
        B.quantize_pack(x, bits, offs, packed, header, 21, 4, 16)
        B.unpack_dequantize(packed, header, bits, offs, out)

    def fill(k):
        scale = np.exp(rng.normal(0, 1.5, (N, 1))).astype(np.float32)
        x.copy_(torch.from_numpy(np.maximum(rng.standard_normal((N, D)).astype(np.float32), 0) * scale))

    fill(0)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        step()                               # warm-up on the capture stream
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        step()
    for k in range(1, 4):
        fill(k)
        graph.replay()
        torch.cuda.synchronize()
        got = (bits.clone(), packed.clone(), header.clone(), out.clone(), res.clone())
        packed.fill_(0xA5)
        out.fill_(float("nan"))
        step()                               # eager, same data
        torch.cuda.synchronize()
        total = int(res[0])
        for a, b in zip(got, (bits, packed[:total], header, out, res)):
            assert torch.equal(a[:total] if a.numel() == packed.numel() else a, b), k
        assert len(set(bits.cpu().tolist())) > 1 and int(res[1]) == 0


# ----------------------------------------------------------------------------- beyond 32-bit indices

def test_element_indices_and_byte_offsets_beyond_32_bits():
    """fp16 [3, 2^30]: element indices run past 2^32 and the bit stream past 2^31 bytes.  The tensor
    is generated on the GPU; groups sampled at the ends and in the middle of every sample are pulled
    back and compared, bit for bit, with the oracle's single-group routines."""
    N, D = 3, 1 << 30
    ng = D // 256
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev).manual_seed(123)
    x = torch.empty((N, D), dtype=torch.float16, device=dev)
    for n in range(N):
        x[n].normal_(0, 1.5, generator=gen)
    bits_np = np.array([8, 8, 4], dtype=np.uint8)
    offsets_np, total = B.packed_bytes(N, D, bits_np)
    assert int(offsets_np[2]) == 1 << 31 and total == (1 << 31) + (1 << 29)
    bits = torch.from_numpy(bits_np).to(dev)
    offsets = torch.from_numpy(offsets_np.view(np.int64)).to(dev)
    packed = torch.full((total + 256,), 0xA5, dtype=torch.uint8, device=dev)
    header = torch.full((N * ng * 2 + 64,), float("nan"), dtype=torch.float32, device=dev)
    gmin = torch.empty((N, ng), dtype=torch.float32, device=dev)
    grange = torch.empty((N, ng), dtype=torch.float32, device=dev)
    out = torch.full((N * D + 64,), float("nan"), dtype=torch.float16, device=dev)
    seed, tag = 0x1234567890, 17
    print("[2^30 features] launching", flush=True)
    B.group_stats(x, gmin, grange)
    B.quantize_pack(x, bits, offsets, packed[:total], header[:N * ng * 2], seed, tag, 16)
    B.unpack_dequantize(packed[:total], header[:N * ng * 2], bits, offsets, out[:N * D].view(N, D))
    torch.cuda.synchronize()
    assert (packed[total:] == 0xA5).all() and torch.isnan(header[N * ng * 2:]).all() and torch.isnan(out[N * D:]).all()
    rng = np.random.default_rng(0)
    picks = [0, 1, 2, 3, 4, ng // 2 - 1, ng // 2, ng - 5, ng - 4, ng - 3, ng - 2, ng - 1] + list(rng.integers(0, ng, 12))
    hd = header[:N * ng * 2].view(N, ng, 2)
    outv = out[:N * D].view(N, D)
    for n in range(N):
        b = int(bits_np[n])
        for g in picks:
            g = int(g)
            xg = x[n, g * 256:(g + 1) * 256].cpu().numpy()
            want_bytes, want_hd = oracle.quantize_group(xg, b, seed, tag, n, g * 256, noise_bits=16)
            lo = int(offsets_np[n]) + g * 32 * b
            assert np.array_equal(packed[lo:lo + 32 * b].cpu().numpy(), want_bytes), (n, g)
            assert np.array_equal(hd[n, g].cpu().numpy().view(np.uint32), want_hd.view(np.uint32)), (n, g)
            omin, orange = oracle.group_stats(xg.reshape(1, 256))
            assert gmin[n, g].item() == omin[0, 0] and grange[n, g].item() == orange[0, 0]
            want_out = oracle.dequantize_group(want_bytes, want_hd, b, 256, out_dtype=np.float16)
            assert np.array_equal(outv[n, g * 256:(g + 1) * 256].cpu().numpy().view(np.uint16), want_out.view(np.uint16)), (n, g)


# ----------------------------------------------------------------------------- full sizes

def _full_size(wl, noise_bits, out_dtype):
    print(f"[full-size] {wl.name} noise_bits={noise_bits}", flush=True)
    x = synth.make_input(wl)
    _round_trip(x.reshape(wl.N, wl.D), wl.bits, wl.philox_seed, wl.tag, noise_bits, (out_dtype,))


def test_config2_r50_stage1_full_size():
    _full_size(synth.r50_stage1(), 24, torch.float32)


def test_config2_r50_stage1_full_size_noise16():
    _full_size(synth.r50_stage1(), 16, torch.float32)


def test_config3_r50_stem_f16_full_size():
    wl = synth.r50_stem_f16()
    x = synth.make_input(wl)
    x2 = x.reshape(wl.N, wl.D)
    gmin, grange = oracle.group_stats(x2[:4])
    assert (grange == 0).any(), "the workload must contain zero-range groups"
    _round_trip(x2, wl.bits, wl.philox_seed, wl.tag, 24, (torch.float16,))


@pytest.mark.parametrize("variant", [0, 1])
def test_config4_fpn_full_size(variant):
    _full_size(synth.fpn(variant), 24, torch.float32)


SWEEP_CHUNKS = 9


@pytest.mark.parametrize("chunk", range(SWEEP_CHUNKS))
def test_config5_resnet50_sweep_batch256(chunk):
    """All 53 tensors at batch 256: widths from actq_allocate_bits (2.0-bit average budget over
    the whole network), then every layer through quantize -> dequantize with a full
    element-by-element comparison (inputs generated on the GPU, copied back for the oracle).
    The 53 layers are spread over several test cases only to keep each case short."""
    shapes = synth.resnet50_conv_input_shapes()
    N = 256
    Dl = np.array([c * h * w for c, h, w in shapes], dtype=np.int64)
    w = synth.lognormal_sensitivities(N * len(shapes), seed=5)
    Dall = np.repeat(Dl, N)
    budget = 2 * int(Dall.sum())
    bits_all = B.allocate_bits(w, Dall, budget)
    if chunk == 0:
        assert np.array_equal(bits_all, oracle.allocate_bits(w, Dall, budget))
    gen = torch.Generator(device="cuda:0")
    for l in range(chunk, len(shapes), SWEEP_CHUNKS):
        D = int(Dl[l])
        gen.manual_seed(1000 + l)
        xt = torch.randn((N, D), generator=gen, device="cuda:0", dtype=torch.float32).clamp_min_(0)
        x = xt.cpu().numpy()
        del xt
        _round_trip(x, bits_all[l * N:(l + 1) * N], seed=15, tag=l, noise_bits=24)


# ----------------------------------------------------------------------------- accepted sides of the argument limits

def test_arguments_exactly_at_their_limits_are_accepted():
    """The host-only tests can only show that a call beyond a limit is refused; here the calls
    exactly at the limits go through and give the oracle's results."""
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(12)
    # a stream buffer of exactly one bit per element with every width 1, D with one element in the last group
    N, D = 3, 2 * 256 + 1
    x_np = rng.standard_normal((N, D)).astype(np.float32)
    bits_np = np.ones(N, dtype=np.uint8)
    off_np, total = B.packed_bytes(N, D, bits_np)
    assert total == N * 3 * 32
    x = torch.from_numpy(x_np).to(dev)
    bits = torch.from_numpy(bits_np).to(dev)
    offs = torch.from_numpy(off_np.view(np.int64)).to(dev)
    buf = torch.full((total + 64,), 0xA5, dtype=torch.uint8, device=dev)
    header = torch.empty(N * 3 * 2, dtype=torch.float32, device=dev)
    for noise_bits in (16, 24):                         # the two accepted values
        B.quantize_pack(x, bits, offs, buf[:total], header, seed=3, tag=1, noise_bits=noise_bits)
        torch.cuda.synchronize()
        opacked, oheader, _ = oracle.quantize_pack(x_np, bits_np, 3, 1, noise_bits=noise_bits)
        assert np.array_equal(buf[:total].cpu().numpy(), opacked) and (buf[total:] == 0xA5).all()
        assert np.array_equal(header.cpu().numpy().view(np.uint32), oheader.reshape(-1).view(np.uint32))
    # one tensor in a multi-tensor call (the smallest count)
    xm_np = rng.standard_normal((N, 512)).astype(np.float32)
    o2, t2 = B.packed_bytes(N, 512, bits_np)
    entry = {"x": torch.from_numpy(xm_np).to(dev), "out": torch.empty((N, 512), device=dev),
             "gmin": torch.empty((N, 2), device=dev), "grange": torch.empty((N, 2), device=dev),
             "header": torch.empty(N * 2 * 2, device=dev), "bits": bits,
             "offsets": torch.from_numpy(o2.view(np.int64)).to(dev), "D": 512}
    table = B.tensor_table([entry])
    pk = torch.zeros(t2, dtype=torch.uint8, device=dev)
    B.group_stats_multi(table, B.ACTQ_F32, N)
    B.quantize_pack_multi(table, B.ACTQ_F32, N, pk, seed=3, tag=7, noise_bits=16)
    torch.cuda.synchronize()
    omin, orange = oracle.group_stats(xm_np)
    assert np.array_equal(entry["gmin"].cpu().numpy().view(np.uint32), omin.view(np.uint32))
    assert np.array_equal(pk.cpu().numpy(), oracle.quantize_pack(xm_np, bits_np, 3, 7, noise_bits=16)[0])
    # device allocator: a budget of zero is a valid argument (status: infeasible, narrowest widths);
    # with per-item sizes the common size is ignored, whatever it is
    M = 5
    w = torch.from_numpy(rng.lognormal(0, 1, M).astype(np.float32)).to(dev)
    D_items_np = np.array([1, 255, 256, 257, 1024], dtype=np.int64)
    D_items = torch.from_numpy(D_items_np).to(dev)
    got_bits = torch.empty(M, dtype=torch.uint8, device=dev)
    got_offs = torch.empty(M, dtype=torch.int64, device=dev)
    res = torch.empty(2, dtype=torch.int64, device=dev)
    B.allocate_bits_device(w, D_items, 0, B.ACTQ_WIDTHS_ALL, got_bits, got_offs, res)
    torch.cuda.synchronize()
    assert int(res[1]) == B.ACTQ_EINFEASIBLE and (got_bits == 1).all()
    budget = int(3 * D_items_np.sum())
    B.allocate_bits_device(w, D_items, budget, B.ACTQ_WIDTHS_ALL, got_bits, got_offs, res)
    torch.cuda.synchronize()
    want = oracle.allocate_bits(w.cpu().numpy(), D_items_np, budget, oracle.WIDTHS_ALL)
    assert int(res[1]) == 0 and np.array_equal(got_bits.cpu().numpy(), want)
    # one item of one element, and a tensor of one element
    one = torch.ones(1, dtype=torch.float32, device=dev)
    B.allocate_bits_device(one, 1, 4, B.ACTQ_WIDTHS_POW2, got_bits[:1], got_offs[:1], res)
    torch.cuda.synchronize()
    assert int(res[1]) == 0 and int(got_bits[0]) == 4 and int(res[0]) == 32 * 4
    zr = B.tensor_stats(torch.full((16,), 2.5, device=dev)[:1].contiguous())
    torch.cuda.synchronize()
    assert zr.cpu().tolist() == [2.5, 0.0]


# statistics of single tensors up to 144 MiB load through the caches, larger ones do not: both against the extremes themselves, whole
# groups, one element in the last group, and rows that begin off the loads' alignment
@pytest.mark.parametrize("dtype", [torch.float32, torch.float16])
@pytest.mark.parametrize("tail", [0, 1, 255])
@pytest.mark.parametrize("over", [False, True])
def test_statistics_on_both_sides_of_the_cached_size(over, tail, dtype):
    N, size = 8, torch.finfo(dtype).bits // 8
    groups = (144 << 20) // (size * N * 256)
    D = (groups + over) * 256 - (256 - tail if tail else 0)
    assert (N * D * size > 144 << 20) == over
    g = torch.Generator(device="cuda").manual_seed(tail + 2 * over)
    x = torch.randn((N, D), generator=g, device="cuda").to(dtype)
    gmin, grange = B.group_stats(x)
    full = torch.cat([x, x[:, -1:].expand(N, -D % 256)], 1).view(N, -1, 256).float()    # the last group repeats its last element
    low = full.amin(2)
    assert torch.equal(gmin, low) and torch.equal(grange, full.amax(2) - low)
