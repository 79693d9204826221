"""Parity of the exact layer contexts (ReLU bit mask, max-pooling positions) with the oracle,
through the C ABI.  Everything is compared bit for bit: masks, positions, outputs, gradients."""
import numpy as np
import pytest
import torch

import oracle
from paper_2104_14129_amd import binding as B

pytestmark = pytest.mark.gpu

CANARY = 0xA5
NP = {np.float32: torch.float32, np.float16: torch.float16}


def _bits_equal(a, b):
    return np.array_equal(np.ascontiguousarray(a).view(np.uint8), np.ascontiguousarray(b).view(np.uint8))


def _relu_round_trip(x_np, g_np, in_place=False):
    n = x_np.size
    dev = torch.device("cuda:0")
    pad = 64
    xbuf = torch.full((n + pad,), 7.0, dtype=NP[x_np.dtype.type], device=dev)
    xbuf[:n] = torch.from_numpy(x_np.reshape(-1)).to(dev)
    x = xbuf[:n]
    mbytes = B.relu_mask_bytes(n)
    mbuf = torch.full((mbytes + 256,), CANARY, dtype=torch.uint8, device=dev)
    ybuf = xbuf if in_place else torch.full((n + pad,), float("nan"), dtype=x.dtype, device=dev)
    B.relu_forward(x, ybuf[:n], mbuf[:mbytes])
    torch.cuda.synchronize()
    oy, omask = oracle.relu_forward(x_np.reshape(-1))
    assert (mbuf[mbytes:] == CANARY).all(), "relu_forward wrote past the mask"
    if in_place:
        assert (xbuf[n:] == 7.0).all()
    else:
        assert torch.isnan(ybuf[n:]).all(), "relu_forward wrote past y"
    assert np.array_equal(mbuf[:mbytes].cpu().numpy(), omask)
    assert _bits_equal(ybuf[:n].cpu().numpy(), oy)
    gbuf = torch.full((n + pad,), float("nan"), dtype=x.dtype, device=dev)
    gy = torch.from_numpy(g_np.reshape(-1)).to(dev)
    if in_place:
        gbuf[:n] = gy
        B.relu_backward(mbuf[:mbytes], gbuf[:n], gbuf[:n])
    else:
        B.relu_backward(mbuf[:mbytes], gy, gbuf[:n])
    torch.cuda.synchronize()
    assert torch.isnan(gbuf[n:]).all(), "relu_backward wrote past grad_x"
    assert _bits_equal(gbuf[:n].cpu().numpy(), oracle.relu_backward(omask, g_np.reshape(-1)))


@pytest.mark.parametrize("dtype", [np.float32, np.float16])
@pytest.mark.parametrize("n", [1, 3, 255, 256, 257, 1023, 1024, 1025, 2047, 2048, 2049, 4096 * 5, 4096 * 37 + 1999])
def test_relu_sizes_spanning_tiles_and_ragged_tails(n, dtype):
    rng = np.random.default_rng(n)
    x = rng.standard_normal(n).astype(dtype)
    x[rng.integers(0, n, n // 7 + 1)] = 0.0
    x[rng.integers(0, n, n // 9 + 1)] = -0.0
    g = rng.standard_normal(n).astype(dtype)
    _relu_round_trip(x, g)
    _relu_round_trip(x, g, in_place=True)


def test_relu_special_values_and_negative_gradients():
    x = np.array([-0.0, 0.0, -np.inf, np.inf, 1e-45, -1e-45, 3.0, -3.0] * 40, dtype=np.float32)
    g = np.array([-1, 2, -3, -np.inf, 5, -6, -7, -8] * 40, dtype=np.float32)
    _relu_round_trip(x, g)
    _relu_round_trip(x.astype(np.float16), g.astype(np.float16))


def test_relu_stem_size():
    """ReLU after the ResNet-50 stem at batch 32: fp32 [32,64,112,112]."""
    rng = np.random.default_rng(1)
    x = rng.standard_normal((32, 64, 112, 112), dtype=np.float32)
    g = rng.standard_normal((32, 64, 112, 112), dtype=np.float32)
    _relu_round_trip(x, g)


CONFIGS = [
    # planes-shape, H, W, kernel, stride, padding, dilation
    ((2, 3), 112, 112, (3, 3), (2, 2), (1, 1), (1, 1)),
    ((5,), 8, 8, (2, 2), (2, 2), (0, 0), (1, 1)),
    ((3,), 9, 11, (3, 2), (1, 2), (1, 0), (2, 1)),
    ((4,), 7, 5, (1, 1), (1, 1), (0, 0), (1, 1)),
    ((2, 2), 13, 17, (5, 4), (3, 2), (2, 2), (1, 2)),
    ((1,), 16, 16, (16, 16), (1, 1), (0, 0), (1, 1)),
    ((7,), 6, 6, (3, 3), (1, 1), (1, 1), (1, 1)),
    ((1, 1), 1, 1, (1, 1), (1, 1), (0, 0), (1, 1)),
    ((3,), 33, 65, (3, 3), (2, 2), (1, 1), (1, 1)),
    ((2,), 40, 37, (7, 5), (5, 3), (3, 2), (1, 1)),
    ((2,), 29, 31, (4, 6), (7, 6), (2, 3), (3, 2)),
    ((70000,), 4, 4, (2, 2), (2, 2), (0, 0), (1, 1)),
    ((3,), 12, 16, (3, 3), (1, 1), (1, 1), (1, 1)),     # fast path, stride 1
    ((3,), 11, 13, (2, 2), (1, 1), (1, 1), (1, 1)),
    ((3,), 14, 20, (2, 2), (2, 2), (1, 1), (1, 1)),
    ((3,), 15, 19, (3, 3), (2, 2), (0, 0), (1, 1)),
    ((2,), 17, 24, (3, 3), (2, 2), (1, 0), (1, 1)),
    ((5,), 12, 16, (3, 3), (2, 2), (1, 1), (1, 1)),     # two outputs per lane
    ((5,), 9, 4, (3, 3), (2, 2), (1, 1), (1, 1)),
    ((3,), 10, 36, (2, 2), (2, 2), (0, 0), (1, 1)),
    ((3,), 7, 8, (3, 3), (2, 2), (0, 1), (1, 1)),
    ((4,), 11, 24, (3, 3), (2, 2), (1, 1), (1, 1)),     # eight inputs per lane in the backward pass
    ((4,), 6, 32, (2, 2), (2, 2), (0, 0), (1, 1)),
    ((2,), 5, 8, (3, 3), (2, 2), (1, 1), (1, 1)),
    ((3,), 6, 520, (3, 3), (2, 2), (1, 1), (1, 1)),     # flattened rows: longer than a wavefront covers
    ((3,), 4, 264, (2, 2), (2, 2), (0, 0), (1, 1)),
    ((7,), 2, 8, (3, 3), (2, 2), (1, 1), (1, 1)),       # one output row per plane: first and last at once
    ((9,), 10, 24, (3, 3), (2, 2), (1, 1), (1, 1)),     # lanes of one wavefront in several planes
     # more planes than one grid dimension holds
]


def _pool_round_trip(x_np, g_np, H, W, k, s, p, d):
    dev = torch.device("cuda:0")
    x = torch.from_numpy(x_np).to(dev)
    oy, oarg = oracle.maxpool2d_forward(x_np, k, s, p, d)
    nout = oy.size
    ybuf = torch.full((nout + 64,), float("nan"), dtype=x.dtype, device=dev)
    abuf = torch.full((nout + 64,), CANARY, dtype=torch.uint8, device=dev)
    y, arg = B.maxpool2d_forward(x, k, s, p, d, ybuf[:nout].view(oy.shape), abuf[:nout].view(oy.shape))
    torch.cuda.synchronize()
    assert torch.isnan(ybuf[nout:]).all() and (abuf[nout:] == CANARY).all()
    assert np.array_equal(arg.cpu().numpy(), oarg)
    assert _bits_equal(y.cpu().numpy(), oy)
    gy = torch.from_numpy(g_np).to(dev)
    gbuf = torch.full((x_np.size + 64,), float("nan"), dtype=x.dtype, device=dev)
    gx = B.maxpool2d_backward(arg, gy, H, W, k, s, p, d, gbuf[:x_np.size].view(x_np.shape))
    torch.cuda.synchronize()
    assert torch.isnan(gbuf[x_np.size:]).all()
    want = oracle.maxpool2d_backward(oarg, g_np, H, W, k, s, p, d)
    assert _bits_equal(gx.cpu().numpy(), want)


# rows of every remainder of a lane's 4 or 8 columns and 2, 4 or 8 outputs, odd and even extents, one-row and one-column
# images, wavefronts that end in the middle of a row, several planes per wavefront, the tensor's last wavefront
ROW_SHAPES = [((3,), 1, 1), ((5,), 1, 9), ((4,), 9, 1), ((2,), 3, 3), ((7,), 5, 6), ((3,), 8, 7), ((2, 3), 17, 8), ((3,), 16, 9), ((3,), 6, 10),
              ((2,), 7, 11), ((3,), 4, 12), ((2,), 9, 13), ((2,), 10, 14), ((3,), 11, 15), ((3,), 12, 17), ((1,), 57, 57), ((3,), 33, 131),
              ((2,), 5, 515), ((130,), 7, 7)]


@pytest.mark.parametrize("dtype", [np.float32, np.float16])
@pytest.mark.parametrize("k,s,p", [(3, 2, 1), (3, 2, 0), (2, 2, 0), (3, 1, 1)])
@pytest.mark.parametrize("shape", ROW_SHAPES)
def test_maxpool_rows_of_any_extent(shape, k, s, p, dtype):
    lead, H, W = shape
    if H + 2 * p < k or W + 2 * p < k:
        pytest.skip("the window does not fit")
    rng = np.random.default_rng(H * 1000 + W)
    # few values: many ties, which the first of a window wins, also at the padded edges; the lowest values there are
    x = rng.integers(-3, 3, lead + (H, W)).astype(dtype)
    x[rng.random(x.shape) < 0.1] = np.finfo(dtype).min
    x[rng.random(x.shape) < 0.1] = -0.0
    x[rng.random(x.shape) < 0.1] = np.finfo(dtype).smallest_subnormal
    OH, OW = (H + 2 * p - k) // s + 1, (W + 2 * p - k) // s + 1
    g = rng.standard_normal(lead + (OH, OW)).astype(dtype)
    _pool_round_trip(x, g, H, W, (k, k), (s, s), (p, p), (1, 1))


# padding along one axis: only above and below (2x2), only beside (3x3)
@pytest.mark.parametrize("dtype", [np.float32, np.float16])
@pytest.mark.parametrize("k,p", [(3, (0, 1)), (2, (1, 0))])
@pytest.mark.parametrize("shape", ROW_SHAPES + [((5,), 8, 8), ((3,), 16, 24), ((3,), 9, 12), ((2,), 6, 56), ((3,), 6, 520)])
def test_maxpool_rows_padded_along_one_axis(shape, k, p, dtype):
    lead, H, W = shape
    if H + 2 * p[0] < k or W + 2 * p[1] < k:
        pytest.skip("the window does not fit")
    rng = np.random.default_rng(H * 1000 + W)
    x = rng.integers(-3, 3, lead + (H, W)).astype(dtype)
    x[rng.random(x.shape) < 0.1] = np.finfo(dtype).min
    x[rng.random(x.shape) < 0.1] = -0.0
    g = rng.standard_normal(lead + ((H + 2 * p[0] - k) // 2 + 1, (W + 2 * p[1] - k) // 2 + 1)).astype(dtype)
    _pool_round_trip(x, g, H, W, (k, k), (2, 2), p, (1, 1))


@pytest.mark.parametrize("k,p,like", [(3, (0, 1), (1, 1)), (2, (1, 0), (0, 0))])
def test_maxpool_padded_along_one_axis_takes_no_longer(k, p, like):
    """The same traffic as the evenly padded window (binary16, 103 MB): with one output per lane it takes 1.9 to 2.8 times as long."""
    x = torch.randn((4096, 112, 112), device="cuda:0").half()
    def us(pad):
        y, arg = B.maxpool2d_forward(x, (k, k), (2, 2), pad)
        times = []
        for _ in range(15):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            B.maxpool2d_forward(x, (k, k), (2, 2), pad, (1, 1), y, arg)
            b.record()
            b.synchronize()
            times.append(a.elapsed_time(b))
        return sorted(times)[7]
    us(p)
    assert us(p) < 1.4 * us(like)


def test_maxpool_with_more_planes_than_a_launch_has_lanes():
    """2^31 + 5 planes of one element: each is its own maximum, at the centre of its window."""
    n = (1 << 31) + 5
    x = torch.arange(-97, 98, device="cuda:0").half().repeat(n // 195 + 1)[:n].view(n, 1, 1)
    y, arg = B.maxpool2d_forward(x, (3, 3), (2, 2), (1, 1))
    assert torch.equal(y, x) and int(arg.min()) == 4 and int(arg.max()) == 4
    y.fill_(float("nan"))
    assert torch.equal(B.maxpool2d_backward(arg, x, 1, 1, (3, 3), (2, 2), (1, 1), grad_x=y), x)


def test_maxpool_beyond_2_to_the_31_lanes_takes_no_longer():
    """binary16, 34 GB: twice the traffic of half the planes.  With a lane per element it takes six times as long."""
    planes, some = (1 << 31) // (112 * 14) + 3, 1024
    part = torch.randn((some, 112, 112), device="cuda:0").half()
    x = part.repeat((planes + some - 1) // some, 1, 1)[:planes]
    window = (3, 3), (1, 1), (1, 1)
    y, arg = torch.empty_like(x), torch.empty(x.shape, dtype=torch.uint8, device="cuda:0")
    def ms(call):
        times = []
        for _ in range(4):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            call()
            b.record()
            b.synchronize()
            times.append(a.elapsed_time(b))
        return min(times)
    forward = lambda n: ms(lambda: B.maxpool2d_forward(x[:n], *window, (1, 1), y[:n], arg[:n]))
    half, whole = forward(planes // 2), forward(planes)
    want, codes = B.maxpool2d_forward(part, *window)
    places = [(0, some)] + [(k * some, some) for k in (planes // 2 // some, planes // 2 // some + 1)] + [(planes // some * some, planes % some)]
    for at, count in places:
        assert torch.equal(y[at:at + count], want[:count]) and torch.equal(arg[at:at + count], codes[:count])
    backward = lambda n: ms(lambda: B.maxpool2d_backward(arg[:n], x[:n], 112, 112, *window, grad_x=y[:n]))
    half_back, whole_back = backward(planes // 2), backward(planes)
    want = B.maxpool2d_backward(codes, part, 112, 112, *window)
    for at, count in places:
        assert torch.equal(y[at:at + count], want[:count])
    assert whole < 2.6 * half and whole_back < 2.6 * half_back, (half, whole, half_back, whole_back)


# rows of whole groups of four and of eight, whole 32 and 64 bytes, over even and odd heights
@pytest.mark.parametrize("dtype", [np.float32, np.float16])
@pytest.mark.parametrize("k,s,p", [(3, 2, 1), (3, 2, 0), (2, 2, 0), (3, 1, 1)])
@pytest.mark.parametrize("shape", [((5,), 8, 8), ((3,), 16, 24), ((3,), 9, 12), ((2,), 7, 20), ((7,), 4, 16), ((3,), 5, 32), ((2,), 6, 56)])
def test_maxpool_aligned_rows(shape, k, s, p, dtype):
    test_maxpool_rows_of_any_extent(shape, k, s, p, dtype)


# The backward kernels and their stores depend on the size of the result and on the length and alignment of a row.
@pytest.mark.parametrize("dtype,planes,H,W,k,s,p", [
    (torch.float16, 2752, 112, 112, 3, 2, 1), (torch.float16, 8256, 64, 64, 3, 2, 1), (torch.float16, 8400, 63, 64, 3, 2, 1),
    (torch.float16, 40, 56, 1000, 3, 2, 1), (torch.float16, 1200, 24, 24, 3, 2, 1), (torch.float16, 2600, 16, 16, 3, 2, 1),
    (torch.float16, 8256, 64, 64, 3, 2, 0), (torch.float16, 8256, 64, 64, 3, 1, 1), (torch.float16, 2752, 112, 112, 2, 2, 0),
    (torch.float16, 10752, 112, 112, 2, 2, 0), (torch.float32, 10560, 40, 40, 3, 2, 0), (torch.float32, 10560, 41, 40, 3, 2, 1),
    (torch.float32, 8208, 64, 64, 2, 2, 0), (torch.float32, 21440, 56, 56, 2, 2, 0), (torch.float32, 21504, 57, 56, 2, 2, 0),
    (torch.float16, 48, 64, 64, 2, 2, 0), (torch.float16, 40, 32, 1000, 2, 2, 0), (torch.float32, 40, 32, 1000, 2, 2, 0),
    (torch.float16, 32, 12, 224, 2, 2, 0), (torch.float32, 32, 12, 112, 2, 2, 0), (torch.float32, 21504, 48, 48, 2, 2, 0),
    (torch.float32, 21504, 49, 48, 2, 2, 0), (torch.float16, 32768, 56, 56, 2, 2, 0), (torch.float32, 16384, 60, 60, 2, 2, 0),
    (torch.float16, 4096, 200, 200, 2, 2, 0), (torch.float16, 5000, 56, 56, 2, 2, 0), (torch.float16, 450, 32, 1000, 2, 2, 0),
    (torch.float16, 5000, 57, 56, 2, 2, 0), (torch.float32, 5000, 33, 40, 2, 2, 0), (torch.float32, 1500, 225, 225, 3, 2, 1),
    (torch.float32, 6158, 113, 113, 2, 2, 0), (torch.float32, 500, 114, 114, 2, 2, 0), (torch.float16, 12000, 113, 113, 2, 2, 0)])
def test_maxpool_gradients_over_sizes_and_row_lengths(dtype, planes, H, W, k, s, p):
    """Against the oracle on planes of the beginning, the middle and the end; few values, so that there are many ties."""
    x = torch.randn((planes, H, W), device="cuda:0").to(dtype).mul_(4).round_()
    y, arg = B.maxpool2d_forward(x, (k, k), (s, s), (p, p))
    g = torch.randn(y.shape, device="cuda:0").to(dtype)
    gx = B.maxpool2d_backward(arg, g, H, W, (k, k), (s, s), (p, p))
    for at in (0, planes // 2, planes - 4):
        part = slice(at, at + 4)
        oy, oarg = oracle.maxpool2d_forward(x[part].cpu().numpy(), (k, k), (s, s), (p, p))
        assert _bits_equal(y[part].cpu().numpy(), oy) and np.array_equal(arg[part].cpu().numpy(), oarg)
        want = oracle.maxpool2d_backward(oarg, g[part].cpu().numpy(), H, W, (k, k), (s, s), (p, p))
        assert _bits_equal(gx[part].cpu().numpy(), want)
    # every gradient went to exactly one input where windows do not overlap
    if k == s:
        assert torch.equal((gx != 0).sum(), (g != 0).sum())


@pytest.mark.parametrize("dtype", [torch.float32, torch.float16])
@pytest.mark.parametrize("shape,k,s,p", [((2, 57, 57), 3, 2, 1), ((3, 30, 31), 3, 2, 0), ((2, 28, 27), 2, 2, 0), ((2, 19, 21), 3, 1, 1),
                                         ((2, 16, 16), 3, 2, 1), ((2, 16, 24), 2, 2, 0)])
def test_maxpool_at_any_element_address(shape, k, s, p, dtype):
    """Tensors, positions and gradients that start one element (one byte) past an aligned address give what aligned ones give."""
    def shifted(t):
        buf = torch.full((t.numel() + 9,), 7, dtype=t.dtype, device="cuda:0")
        buf[1:1 + t.numel()] = t.reshape(-1)
        return buf, buf[1:1 + t.numel()].view(t.shape)
    x = torch.randn(shape, device="cuda:0").to(dtype)
    y, arg = B.maxpool2d_forward(x, (k, k), (s, s), (p, p))
    g = torch.randn(y.shape, device="cuda:0").to(dtype)
    gx = B.maxpool2d_backward(arg, g, shape[-2], shape[-1], (k, k), (s, s), (p, p))
    ybuf, y1 = shifted(torch.zeros_like(y))
    abuf, a1 = shifted(torch.zeros_like(arg))
    gbuf, gx1 = shifted(torch.zeros_like(x))
    B.maxpool2d_forward(shifted(x)[1], (k, k), (s, s), (p, p), (1, 1), y1, a1)
    B.maxpool2d_backward(a1, shifted(g)[1], shape[-2], shape[-1], (k, k), (s, s), (p, p), (1, 1), gx1)
    assert torch.equal(y1, y) and torch.equal(a1, arg) and torch.equal(gx1, gx)
    for buf in (ybuf, abuf, gbuf):
        assert buf[0] == 7 and (buf[-8:] == 7).all()


@pytest.mark.parametrize("dtype", [np.float32, np.float16])
@pytest.mark.parametrize("cfg", CONFIGS)
def test_maxpool_configs(cfg, dtype):
    lead, H, W, k, s, p, d = cfg
    rng = np.random.default_rng(H * 100 + W)
    x = rng.standard_normal(lead + (H, W)).astype(dtype)
    OH, OW = oracle.pool2d_output_size(H, W, k, s, p, d)
    assert B.pool2d_output_size(H, W, k, s, p, d) == (OH, OW)
    g = rng.standard_normal(lead + (OH, OW)).astype(dtype)
    _pool_round_trip(x, g, H, W, k, s, p, d)
    # many ties: small integers
    xi = rng.integers(-2, 3, size=lead + (H, W)).astype(dtype)
    _pool_round_trip(xi, g, H, W, k, s, p, d)


def test_maxpool_backward_ignores_positions_outside_the_image():
    x = np.random.default_rng(0).standard_normal((1, 6, 6)).astype(np.float32)
    _, arg = oracle.maxpool2d_forward(x, (3, 3), (2, 2), (1, 1))
    gy = np.ones((1, 3, 3), dtype=np.float32)
    bad = arg.copy()
    bad[0, 0, 0] = 0          # points at the padding
    bad[0, 1, 1] = 200        # outside the window
    gx = B.maxpool2d_backward(torch.from_numpy(bad).cuda(), torch.from_numpy(gy).cuda(), 6, 6, (3, 3), (2, 2), (1, 1))
    good = arg.copy()
    want = oracle.maxpool2d_backward(good, gy, 6, 6, (3, 3), (2, 2), (1, 1))
    got = gx.cpu().numpy()
    assert got.sum() == want.sum() - 2          # exactly the two bad outputs are dropped


def test_maxpool_stem_size():
    """The one max pooling of ResNet-50 at batch 32: fp32 [32,64,112,112], 3x3, stride 2, padding 1."""
    rng = np.random.default_rng(2)
    x = np.maximum(rng.standard_normal((32, 64, 112, 112), dtype=np.float32), 0)   # post-ReLU: many ties at 0
    g = rng.standard_normal((32, 64, 56, 56), dtype=np.float32)
    _pool_round_trip(x, g, 112, 112, (3, 3), (2, 2), (1, 1), (1, 1))


@pytest.mark.parametrize("dtype", [np.float32, np.float16])
def test_maxpool_sees_new_contents_of_the_same_buffers(dtype):
    """The pooling kernels take one column per wavefront through the scalar data path; a second
    call on the same buffers, refilled by another kernel on the same stream, must see the new
    contents (rows longer than a wavefront covers, so that those columns are in use)."""
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(17)
    planes, H, W = 3, 6, 520
    k, s, p = (3, 3), (2, 2), (1, 1)
    OH, OW = B.pool2d_output_size(H, W, k, s, p)
    x = torch.empty((planes, H, W), dtype=NP[dtype], device=dev)
    y = torch.empty((planes, OH, OW), dtype=NP[dtype], device=dev)
    arg = torch.empty((planes, OH, OW), dtype=torch.uint8, device=dev)
    gy = torch.empty((planes, OH, OW), dtype=NP[dtype], device=dev)
    gx = torch.empty((planes, H, W), dtype=NP[dtype], device=dev)
    for round_ in range(3):
        x_np = rng.standard_normal((planes, H, W)).astype(dtype)
        g_np = rng.standard_normal((planes, OH, OW)).astype(dtype)
        staged_x, staged_g = torch.from_numpy(x_np).to(dev), torch.from_numpy(g_np).to(dev)
        x.copy_(staged_x)                       # device-side writes, then the kernels, no synchronisation between
        gy.copy_(staged_g)
        B.maxpool2d_forward(x, k, s, p, (1, 1), y, arg)
        B.maxpool2d_backward(arg, gy, H, W, k, s, p, (1, 1), gx)
        torch.cuda.synchronize()
        oy, oarg = oracle.maxpool2d_forward(x_np, k, s, p)
        assert np.array_equal(arg.cpu().numpy(), oarg), round_
        assert _bits_equal(y.cpu().numpy(), oy), round_
        assert _bits_equal(gx.cpu().numpy(), oracle.maxpool2d_backward(oarg, g_np, H, W, k, s, p)), round_


# ReLU results of 48 to 112 MiB are stored through the caches: the same bits as from halves on the other side of the limits, which go past them, and the same
# pooling of both (aligned rows, the stream kernel with and without joined rows, 2x2, rows of odd length); at the lower end, and above the upper one
@pytest.mark.parametrize("dtype", [torch.float32, torch.float16])
@pytest.mark.parametrize("mib,H,W,k,s,p", [(50, 112, 112, 3, 2, 1), (50, 64, 128, 3, 2, 1), (50, 56, 64, 2, 2, 0), (52, 56, 56, 2, 2, 0), (50, 113, 113, 3, 2, 1),
                                           (50, 31, 45, 3, 2, 0), (50, 57, 60, 3, 1, 1), (120, 56, 56, 3, 1, 1), (160, 16, 16, 2, 2, 0)])
def test_results_stored_through_the_caches_equal_those_that_are_not(mib, H, W, k, s, p, dtype):
    size = torch.finfo(dtype).bits // 8
    planes = (mib << 20) // (size * H * W) // 2 * 2
    whole, half = planes * H * W * size, planes // 2 * H * W * size
    inside = lambda n: 48 << 20 <= n <= 112 << 20
    assert inside(whole) != inside(half)
    g = torch.Generator(device="cuda").manual_seed(H + W)
    x = torch.randn((planes, H, W), generator=g, device="cuda").to(dtype)
    y, mask = B.relu_forward(x)
    z, arg = B.maxpool2d_forward(y, (k, k), (s, s), (p, p))
    gz = torch.randn(z.shape, generator=g, device="cuda").to(dtype)
    gy = B.maxpool2d_backward(arg, gz, H, W, (k, k), (s, s), (p, p))
    assert torch.equal(y, torch.relu(x))
    for part in (slice(0, planes // 2), slice(planes // 2, planes)):
        y2, _ = B.relu_forward(x[part].clone())     # (an aligned address)
        z2, arg2 = B.maxpool2d_forward(y2, (k, k), (s, s), (p, p))
        gy2 = B.maxpool2d_backward(arg2, gz[part], H, W, (k, k), (s, s), (p, p))
        assert torch.equal(y[part], y2) and torch.equal(z[part], z2) and torch.equal(arg[part], arg2) and torch.equal(gy[part], gy2)
    n = x.numel() // 2 // 256 * 256      # whole words of the bit stream
    _, mask2 = B.relu_forward(x.view(-1)[:n])
    assert torch.equal(mask[:n // 8], mask2)


# The row kernels have a second form, chosen by the size of the image, its rows and its type: a tensor of 72 MiB has to agree with its
# pieces of 9 MiB (small calls of any extent are compared with the oracle above).  The whole takes the second form and the pieces the first:
# forward, 3x3 but binary16 without row padding, but binary32 rows whose lanes divide a wavefront and but binary16 3x3/1/1 on odd rows.
# The whole takes the first form and the pieces the second: binary16 gradients at stride 2, binary16 3x3/1/1 gradients on odd rows below
# 32 columns (three lanes to a row of 17 to 23 columns, so that rows cross wavefronts; one, two and four lanes do not) and binary32 ones of
# rows whose lanes divide a wavefront.  Elsewhere both take the same form, at other places of the tensor.
# Planes smaller than a workgroup, rows of one and of many wavefronts, and tensors that start between words.
@pytest.mark.parametrize("dtype", [torch.float32, torch.float16])
@pytest.mark.parametrize("k,s,p", [(3, 2, (1, 1)), (3, 2, (0, 0)), (3, 2, (0, 1)), (3, 1, (1, 1))])
@pytest.mark.parametrize("H,W", [(3, 3), (7, 6), (15, 15), (1, 34), (28, 28), (63, 2), (17, 17), (21, 21), (9, 23), (33, 71), (113, 113), (9, 516)])
def test_maxpool_of_large_tensors_equals_that_of_their_pieces(H, W, k, s, p, dtype):
    if H + 2 * p[0] < k or W + 2 * p[1] < k:
        pytest.skip("the window does not fit")
    pieces = 8
    planes = (72 << 20) // (torch.finfo(dtype).bits // 8 * H * W) // pieces * pieces
    gen = torch.Generator(device="cuda").manual_seed(H * 1000 + W)
    x = torch.randint(-3, 4, (planes * H * W + 1,), generator=gen, device="cuda").to(dtype)[1:].view(planes, H, W)   # many ties
    z, arg = B.maxpool2d_forward(x, (k, k), (s, s), p)
    gz = torch.randn(z.shape, generator=gen, device="cuda").to(dtype)
    gx = B.maxpool2d_backward(arg, gz, H, W, (k, k), (s, s), p)
    for i in range(pieces):
        part = slice(i * planes // pieces, (i + 1) * planes // pieces)
        z2, arg2 = B.maxpool2d_forward(x[part], (k, k), (s, s), p)
        assert torch.equal(z[part], z2) and torch.equal(arg[part], arg2), i
        assert torch.equal(gx[part].view(torch.uint8), B.maxpool2d_backward(arg[part], gz[part], H, W, (k, k), (s, s), p).view(torch.uint8)), i
