"""Per-operation parity of the HIP kernels against the fp64 CPU oracle, through
the C ABI, on seeded inputs at sizes that span several tiles and ragged tails."""
import ctypes
import subprocess

import numpy as np
import pytest
import torch

from oracle import vgg_ref as R
from paper_1810_09868_amd import binding as B
from paper_1810_09868_amd import synth

from gpu_util import TDT, TOL, dev, from_nhwc, max_rel_err, to_nhwc, ws_bytes

pytestmark = pytest.mark.gpu

# (N, H, W, Cin, Cout): 2-D patch tiling (H, W multiples of 16), linear tiling with images and rows
# crossing inside a tile, ragged channel counts, a last partial tile, tiny images.
CONV_SHAPES = [
    (2, 32, 32, 64, 128),
    (3, 14, 14, 32, 64),
    (2, 28, 28, 96, 160),
    (3, 5, 7, 3, 20),
    (1, 2, 2, 16, 64),
    (5, 16, 48, 32, 192),
    (1, 56, 56, 64, 64),
    (1, 6, 100, 16, 32),   # wide rows: halo beyond the direct-to-LDS kernels' limit, weight-gradient halo in several batches
    # few tiles and a long contraction: several workgroups share a tile, each with a range of channel
    # chunks (uneven ranges: 9 or 18 chunks of 64 bytes; fp32 only: 5 chunks in two ranges)
    (1, 20, 20, 288, 64),
    (2, 14, 14, 80, 96),
    (1, 14, 14, 512, 512),
]


def _random_conv_shapes(count, seed=11):
    """Seeded shapes that mix the kernels' variants: patch and linear tiles, 64- and 128-wide column tiles,
    odd and even numbers of channel chunks, channel counts off the tile sizes, tiles that cross images."""
    import random
    rnd = random.Random(seed)
    hw = [(5, 7), (16, 16), (17, 16), (28, 28), (30, 33), (56, 56), (14, 14), (32, 48), (9, 100), (64, 64), (2, 2), (112, 16), (3, 130)]
    out = []
    while len(out) < count:
        H, W = rnd.choice(hw)
        N = rnd.choice([1, 2, 3, 5, 9])
        ci = rnd.choice([3, 8, 16, 24, 32, 40, 64, 96, 128, 160])
        co = rnd.choice([8, 20, 64, 72, 128, 136, 192, 256, 320])
        if N * H * W * ci * co * 9 <= 3e9:
            out.append((N, H, W, ci, co))
    return out


RANDOM_CONV_SHAPES = _random_conv_shapes(24)


def _pack(dtype, w, flip=0):
    Cout, Cin = w.shape[:2]
    rows, cols = (Cin, Cout) if flip else (Cout, Cin)
    out = torch.empty((9, rows, B.vgg_padded_channels(dtype, cols)), dtype=TDT[dtype], device="cuda")
    B.vgg_conv_pack_weights(dtype, Cin, Cout, dev(w), out, flip)
    return out


@pytest.mark.parametrize("dtype", [B.F32, B.BF16])
@pytest.mark.parametrize("shape", CONV_SHAPES)
def test_conv3x3_fwd(dtype, shape):
    N, H, W, Cin, Cout = shape
    d = synth.conv_layer_inputs(N, H, W, Cin, Cout, seed=sum(shape))
    ref = R.conv3x3_fwd(d["x"], d["w"], d["b"], relu=True)
    x = to_nhwc(d["x"], dtype)
    y = torch.empty((N, H, W, Cout), dtype=TDT[dtype], device="cuda")
    ws = ws_bytes(B.vgg_conv3x3_fwd_workspace_bytes(dtype, N, H, W, Cin, Cout))
    B.vgg_conv3x3_fwd(dtype, N, H, W, Cin, Cout, x, _pack(dtype, d["w"]), dev(d["b"]), y, 1, ws)
    torch.cuda.synchronize()
    assert max_rel_err(from_nhwc(y), ref) <= TOL[dtype]
    # no bias, no ReLU
    ref2 = R.conv3x3_fwd(d["x"], d["w"], None, relu=False)
    B.vgg_conv3x3_fwd(dtype, N, H, W, Cin, Cout, x, _pack(dtype, d["w"]), None, y, 0, ws)
    torch.cuda.synchronize()
    assert max_rel_err(from_nhwc(y), ref2) <= TOL[dtype]


@pytest.mark.parametrize("dtype", [B.F32, B.BF16])
@pytest.mark.parametrize("shape", [(2, 32, 32, 64, 128), (3, 16, 48, 32, 64), (1, 112, 112, 32, 192)])
def test_conv3x3_fwd_with_fused_pool(dtype, shape):
    N, H, W, Cin, Cout = shape
    d = synth.conv_layer_inputs(N, H, W, Cin, Cout, seed=sum(shape) + 7)
    x = to_nhwc(d["x"], dtype)
    y = torch.full((N, H, W, Cout), float("nan"), dtype=TDT[dtype], device="cuda")
    pooled = torch.full((N, H // 2, W // 2, Cout), float("nan"), dtype=TDT[dtype], device="cuda")
    B.vgg_conv3x3_fwd_pool(dtype, N, H, W, Cin, Cout, x, _pack(dtype, d["w"]), dev(d["b"]), y, pooled, 1)
    torch.cuda.synchronize()
    ref = R.conv3x3_fwd(d["x"], d["w"], d["b"], relu=True)
    pref, _ = R.maxpool2x2(ref)
    assert max_rel_err(from_nhwc(y), ref) <= TOL[dtype]
    assert max_rel_err(from_nhwc(pooled), pref) <= TOL[dtype]
    # the pooled tensor is exactly the 2x2 maximum of what the same launch wrote un-pooled
    pgpu, _ = R.maxpool2x2(from_nhwc(y))
    assert np.array_equal(from_nhwc(pooled), pgpu)
    # un-pooled output suppressed; positions of the maxima requested
    pooled2 = torch.empty_like(pooled)
    arg = torch.full((N, H // 2, W // 2, Cout), 255, dtype=torch.uint8, device="cuda")
    B.vgg_conv3x3_fwd_pool(dtype, N, H, W, Cin, Cout, x, _pack(dtype, d["w"]), dev(d["b"]), None, pooled2, 1, argmax=arg)
    torch.cuda.synchronize()
    assert torch.equal(pooled, pooled2)
    # bit-exact against the first-maximum rule applied to what the launch wrote un-pooled
    _, agpu = R.maxpool2x2(from_nhwc(y))
    assert np.array_equal(arg.permute(0, 3, 1, 2).cpu().numpy(), agpu)
    # and the same bytes as the stand-alone pooling kernel gives
    arg2 = torch.empty_like(arg)
    B.vgg_maxpool2x2(dtype, N, H, W, Cout, y, pooled2, arg2)
    torch.cuda.synchronize()
    assert torch.equal(arg, arg2) and torch.equal(pooled, pooled2)
    with pytest.raises(B.VggError):
        B.vgg_conv3x3_fwd_pool(dtype, N, 14, 14, Cin, Cout, x, _pack(dtype, d["w"]), dev(d["b"]), None, pooled2, 1)


@pytest.mark.parametrize("dtype", [B.F32, B.BF16])
@pytest.mark.parametrize("shape", [(2, 32, 48), (3, 20, 9), (1, 224, 224), (70, 16, 16)])
def test_conv3x3_fwd_first_layer_from_nchw(dtype, shape):
    N, H, W = shape
    d = synth.conv_layer_inputs(N, H, W, 3, 64, seed=sum(shape))
    y = torch.full((N, H, W, 64), float("nan"), dtype=TDT[dtype], device="cuda")
    for relu in (1, 0):
        ref = R.conv3x3_fwd(d["x"], d["w"], d["b"], relu=bool(relu))
        B.vgg_conv3x3_fwd_first(dtype, N, H, W, dev(d["x"]), _pack(dtype, d["w"]), dev(d["b"]), y, relu)
        torch.cuda.synchronize()
        assert max_rel_err(from_nhwc(y), ref) <= TOL[dtype]


@pytest.mark.parametrize("shape", [(1, 16, 32), (2, 32, 64), (3, 48, 32), (22, 64, 128)])
def test_conv3x3_fwd_first_pair(shape):
    """The first two convolutions and the first pool as one call: against the oracle's three operations and
    against the library's separate calls (same products; the first layer adds its 27 in another order, so a
    few values differ by a rounding step).  The pooled tensor must be exactly the 2x2 maximum of the
    un-pooled one.  The last shape has 704 patches, more than the launch's 512 workgroups."""
    N, H, W = shape
    dtype = B.BF16
    d1 = synth.conv_layer_inputs(N, H, W, 3, 64, seed=sum(shape))
    d2 = synth.conv_layer_inputs(1, 4, 4, 64, 64, seed=sum(shape) + 1)
    x = np.abs(d1["x"])      # image-like: non-negative
    b1 = np.linspace(-0.2, 0.3, 64).astype(np.float32)
    b2 = np.linspace(0.1, -0.4, 64).astype(np.float32)
    y1 = R.conv3x3_fwd(x, d1["w"], b1, relu=True)
    y2 = R.conv3x3_fwd(y1, d2["w"], b2, relu=True)
    pooled_ref, _ = R.maxpool2x2(y2)
    w1, w2 = _pack(dtype, d1["w"]), _pack(dtype, d2["w"])
    xd = dev(x.astype(np.float32))
    y2_g = torch.empty((N, H, W, 64), dtype=TDT[dtype], device="cuda")
    po_g = torch.empty((N, H // 2, W // 2, 64), dtype=TDT[dtype], device="cuda")
    B.vgg_conv3x3_fwd_first_pair(dtype, N, H, W, xd, w1, dev(b1), w2, dev(b2), y2_g, po_g)
    torch.cuda.synchronize()
    assert max_rel_err(from_nhwc(y2_g), y2) <= TOL[dtype]
    assert max_rel_err(from_nhwc(po_g), pooled_ref) <= TOL[dtype]
    # pooled == 2x2 maximum of the un-pooled output, bit for bit
    po_chk = torch.empty_like(po_g)
    B.vgg_maxpool2x2(dtype, N, H, W, 64, y2_g, po_chk)
    torch.cuda.synchronize()
    assert torch.equal(po_g.view(torch.int16), po_chk.view(torch.int16))
    # the separate calls: bf16 roundings of slightly different fp32 sums
    y1_s = torch.empty((N, H, W, 64), dtype=TDT[dtype], device="cuda")
    y2_s = torch.empty_like(y2_g)
    po_s = torch.empty_like(po_g)
    B.vgg_conv3x3_fwd_first(dtype, N, H, W, xd, w1, dev(b1), y1_s, 1)
    ws = ws_bytes(B.vgg_conv3x3_fwd_workspace_bytes(dtype, N, H, W, 64, 64))
    B.vgg_conv3x3_fwd_pool(dtype, N, H, W, 64, 64, y1_s, w2, dev(b2), y2_s, po_s, 1, ws)
    torch.cuda.synchronize()
    assert max_rel_err(from_nhwc(y2_g), from_nhwc(y2_s)) <= 2.0 ** -7
    # only one of the two outputs
    po_only = torch.zeros_like(po_g)
    B.vgg_conv3x3_fwd_first_pair(dtype, N, H, W, xd, w1, dev(b1), w2, dev(b2), None, po_only)
    torch.cuda.synchronize()
    assert torch.equal(po_only.view(torch.int16), po_g.view(torch.int16))
    y_only = torch.zeros_like(y2_g)
    B.vgg_conv3x3_fwd_first_pair(dtype, N, H, W, xd, w1, dev(b1), w2, dev(b2), y_only, None)
    torch.cuda.synchronize()
    assert torch.equal(y_only.view(torch.int16), y2_g.view(torch.int16))


def test_conv3x3_fwd_first_pair_rejects_other_shapes_and_dtypes():
    x = torch.zeros((1, 3, 16, 16), device="cuda")
    w = torch.zeros((9 * 64 * 64,), dtype=torch.bfloat16, device="cuda")
    y = torch.zeros((1, 16, 16, 64), dtype=torch.bfloat16, device="cuda")
    L = B.lib()
    args = (x.data_ptr(), w.data_ptr(), None, w.data_ptr(), None, y.data_ptr(), None, None)
    assert L.vgg_conv3x3_fwd_first_pair(B.BF16, 1, 16, 16, *args) == -7      # W not a multiple of 32
    assert L.vgg_conv3x3_fwd_first_pair(B.F32, 1, 16, 32, *args) == -7       # fp32
    assert L.vgg_conv3x3_fwd_first_pair(B.BF16, 1, 16, 32, x.data_ptr(), w.data_ptr(), None, w.data_ptr(), None, None, None, None) == -1


@pytest.mark.parametrize("dtype", [B.F32, B.BF16])
@pytest.mark.parametrize("shape", CONV_SHAPES)
def test_conv3x3_bwd_data(dtype, shape):
    N, H, W, Cin, Cout = shape
    d = synth.conv_layer_inputs(N, H, W, Cin, Cout, seed=sum(shape) + 1)
    ref = R.conv3x3_bwd_data(d["dy"], d["w"])
    g = to_nhwc(d["dy"], dtype)
    dx = torch.empty((N, H, W, Cin), dtype=TDT[dtype], device="cuda")
    ws = ws_bytes(B.vgg_conv3x3_bwd_data_workspace_bytes(dtype, N, H, W, Cin, Cout))
    wtf = _pack(dtype, d["w"], flip=1)
    B.vgg_conv3x3_bwd_data(dtype, N, H, W, Cin, Cout, g, wtf, None, dx, ws)
    torch.cuda.synchronize()
    assert max_rel_err(from_nhwc(dx), ref) <= TOL[dtype]
    # fused ReLU backward of the producer of x: dx * (x > 0)
    xsrc = to_nhwc(d["x"], dtype)
    B.vgg_conv3x3_bwd_data(dtype, N, H, W, Cin, Cout, g, wtf, xsrc, dx, ws)
    torch.cuda.synchronize()
    assert max_rel_err(from_nhwc(dx), ref * (from_nhwc(xsrc) > 0)) <= TOL[dtype]


# The convolution layers of the batch-100 benchmark whose launches take kernels that the small shapes above
# never reach (bf16: weights in registers, with 256- and with 320-pixel tiles).  (N, H, W, Cin, Cout,
# expected kernel of the forward call, expected kernel of the data gradient with a mask.)
FULL_SIZE_LAYERS = [
    (100, 112, 112, 64, 128, 4, 1),
    (100, 56, 56, 128, 256, 5, 5),
    (100, 56, 56, 256, 256, 5, 5),
    (100, 28, 28, 256, 512, 4, 4),
    (100, 28, 28, 512, 512, 4, 4),
    (100, 14, 14, 512, 512, 7, 7),
]


def _sample_pixels(N, H, W, tile_rows, count, seed):
    """Pixels (n, h, w) to check at full size: the tensor's first and last pixels, the corners of an image,
    both sides of the first, a middle and the last tile boundary, and `count` random ones."""
    M = N * H * W
    flat = {0, 1, W - 1, W, H * W - 1, H * W, M - 1, M - W, M - H * W}
    for t in (1, (M // tile_rows) // 2, M // tile_rows):
        for d in (-1, 0, 1):
            flat.add(min(max(t * tile_rows + d, 0), M - 1))
    rng = np.random.default_rng(np.random.PCG64(seed))
    flat.update(int(v) for v in rng.integers(0, M, size=count))
    flat = np.array(sorted(flat))
    return flat // (H * W), (flat % (H * W)) // W, flat % W


def _patches(t_nchw, n, h, w):
    """The zero-padded 3x3 neighbourhoods [S, C, 3, 3] of the pixels (n[i], h[i], w[i])."""
    _, C, H, W = t_nchw.shape
    out = np.zeros((len(n), C, 3, 3), dtype=np.float64)
    for dh in range(3):
        for dw in range(3):
            hh, ww = h + dh - 1, w + dw - 1
            ok = (hh >= 0) & (hh < H) & (ww >= 0) & (ww < W)
            out[ok, :, dh, dw] = t_nchw[n[ok], :, hh[ok], ww[ok]]
    return out


@pytest.mark.parametrize("shape,kernel", [((42, 28, 28, 64, 512), 4), ((11, 56, 56, 64, 512), 5), ((33, 32, 32, 64, 512), 4)])
def test_conv3x3_bf16_weights_in_registers_element_by_element(shape, kernel):
    """The weights-in-registers kernel at sizes the oracle computes whole: just over 512 tiles of 256 pixels x 128
    channels (the smallest launches that take it), consecutive-pixel tiles with both halo sizes and patch tiles.
    Forward (plain stores straight from registers), forward with the fused pool where the size allows it, and
    the data gradient of the mirrored layer with its mask."""
    dtype = B.BF16
    N, H, W, Cin, Cout = shape
    assert B.vgg_conv3x3_plan(B.PLAN_FWD, dtype, N, H, W, Cin, Cout)[0] == kernel
    d = synth.conv_layer_inputs(N, H, W, Cin, Cout, seed=sum(shape))
    ref = R.conv3x3_fwd(d["x"], d["w"], d["b"], relu=True)
    x = to_nhwc(d["x"], dtype)
    wp = _pack(dtype, d["w"])
    y = torch.empty((N, H, W, Cout), dtype=TDT[dtype], device="cuda")
    ws = ws_bytes(B.vgg_conv3x3_fwd_workspace_bytes(dtype, N, H, W, Cin, Cout))
    B.vgg_conv3x3_fwd(dtype, N, H, W, Cin, Cout, x, wp, dev(d["b"]), y, 1, ws)
    torch.cuda.synchronize()
    assert max_rel_err(from_nhwc(y), ref) <= TOL[dtype]
    if H % 16 == 0 and W % 16 == 0:
        assert B.vgg_conv3x3_plan(B.PLAN_FWD_POOL, dtype, N, H, W, Cin, Cout)[0] == kernel
        y2 = torch.empty_like(y)
        po = torch.empty((N, H // 2, W // 2, Cout), dtype=TDT[dtype], device="cuda")
        arg = torch.empty((N, H // 2, W // 2, Cout), dtype=torch.uint8, device="cuda")
        B.vgg_conv3x3_fwd_pool(dtype, N, H, W, Cin, Cout, x, wp, dev(d["b"]), y2, po, 1, ws, argmax=arg)
        torch.cuda.synchronize()
        assert torch.equal(y2.view(torch.int16), y.view(torch.int16))
        po_chk = torch.empty_like(po)
        arg_chk = torch.empty_like(arg)
        B.vgg_maxpool2x2(dtype, N, H, W, Cout, y, po_chk, arg_chk)
        torch.cuda.synchronize()
        assert torch.equal(po.view(torch.int16), po_chk.view(torch.int16)) and torch.equal(arg, arg_chk)
    # data gradient of the layer with the channel counts swapped: the same implicit GEMM on the flipped packing
    assert B.vgg_conv3x3_plan(B.PLAN_BWD_DATA, dtype, N, H, W, Cout, Cin)[0] == kernel
    d = synth.conv_layer_inputs(N, H, W, Cout, Cin, seed=sum(shape) + 1)
    refd = R.conv3x3_bwd_data(d["dy"], d["w"])
    g = to_nhwc(d["dy"], dtype)
    dx = torch.empty((N, H, W, Cout), dtype=TDT[dtype], device="cuda")
    wsd = ws_bytes(B.vgg_conv3x3_bwd_data_workspace_bytes(dtype, N, H, W, Cout, Cin))
    wtf = _pack(dtype, d["w"], flip=1)
    xsrc = to_nhwc(d["x"], dtype)
    B.vgg_conv3x3_bwd_data(dtype, N, H, W, Cout, Cin, g, wtf, xsrc, dx, wsd)
    torch.cuda.synchronize()
    assert max_rel_err(from_nhwc(dx), refd * (from_nhwc(xsrc) > 0)) <= TOL[dtype]


@pytest.mark.parametrize("cout", [200, 196, 132])
def test_conv3x3_bf16_weights_in_registers_ragged_channels(cout):
    """The weights-in-registers kernel with a last column tile that is only partly there: 200 channels (16-byte
    stores, the last 16-channel blocks of the tile missing), 196 (not a multiple of eight: the element-wise
    epilogue) and 132 (four channels into the second tile); 32 input channels make the contraction a single
    chunk.  Forward against the oracle, element by element; nothing may be written past the tensor."""
    dtype = B.BF16
    N, H, W, Cin = 84, 28, 28, 32
    assert B.vgg_conv3x3_plan(B.PLAN_FWD, dtype, N, H, W, Cin, cout)[0] == 4
    d = synth.conv_layer_inputs(N, H, W, Cin, cout, seed=cout)
    ref = R.conv3x3_fwd(d["x"], d["w"], d["b"], relu=True)
    x = to_nhwc(d["x"], dtype)
    wp = _pack(dtype, d["w"])
    n = N * H * W * cout
    buf = torch.full((n + 4096,), -7.0, dtype=TDT[dtype], device="cuda")      # (guard behind the tensor)
    y = buf[:n].view(N, H, W, cout)
    ws = ws_bytes(B.vgg_conv3x3_fwd_workspace_bytes(dtype, N, H, W, Cin, cout))
    B.vgg_conv3x3_fwd(dtype, N, H, W, Cin, cout, x, wp, dev(d["b"]), y, 1, ws)
    torch.cuda.synchronize()
    assert max_rel_err(from_nhwc(y), ref) <= TOL[dtype]
    assert (buf[n:] == -7.0).all()


def test_conv3x3_bf16_320_pixel_tiles_element_by_element():
    """The 320-pixel tiles (one workgroup per compute unit) at a size the oracle computes whole: 84 images of
    14x14 give 52 such tiles x 4 column tiles, tiles that cross image rows and images, and a ragged last tile.
    Forward on 128 -> 512 channels, data gradient (with and without mask) on 512 -> 128, each checked to be
    the launch that takes that kernel."""
    dtype = B.BF16
    N, H, W = 84, 14, 14
    # forward
    Cin, Cout = 128, 512
    assert B.vgg_conv3x3_plan(B.PLAN_FWD, dtype, N, H, W, Cin, Cout)[:2] in ([6, 320], [7, 320])
    d = synth.conv_layer_inputs(N, H, W, Cin, Cout, seed=8414)
    x = to_nhwc(d["x"], dtype)
    y = torch.empty((N, H, W, Cout), dtype=TDT[dtype], device="cuda")
    ws = ws_bytes(B.vgg_conv3x3_fwd_workspace_bytes(dtype, N, H, W, Cin, Cout))
    B.vgg_conv3x3_fwd(dtype, N, H, W, Cin, Cout, x, _pack(dtype, d["w"]), dev(d["b"]), y, 1, ws)
    torch.cuda.synchronize()
    assert max_rel_err(from_nhwc(y), R.conv3x3_fwd(d["x"], d["w"], d["b"], relu=True)) <= TOL[dtype]
    # data gradient
    Cin, Cout = 512, 128
    assert B.vgg_conv3x3_plan(B.PLAN_BWD_DATA, dtype, N, H, W, Cin, Cout)[:2] in ([6, 320], [7, 320])
    d = synth.conv_layer_inputs(N, H, W, Cin, Cout, seed=8415)
    ref = R.conv3x3_bwd_data(d["dy"], d["w"])
    g = to_nhwc(d["dy"], dtype)
    dx = torch.empty((N, H, W, Cin), dtype=TDT[dtype], device="cuda")
    ws = ws_bytes(B.vgg_conv3x3_bwd_data_workspace_bytes(dtype, N, H, W, Cin, Cout))
    wtf = _pack(dtype, d["w"], flip=1)
    B.vgg_conv3x3_bwd_data(dtype, N, H, W, Cin, Cout, g, wtf, None, dx, ws)
    torch.cuda.synchronize()
    assert max_rel_err(from_nhwc(dx), ref) <= TOL[dtype]
    xsrc = to_nhwc(d["x"], dtype)
    B.vgg_conv3x3_bwd_data(dtype, N, H, W, Cin, Cout, g, wtf, xsrc, dx, ws)
    torch.cuda.synchronize()
    assert max_rel_err(from_nhwc(dx), ref * (from_nhwc(xsrc) > 0)) <= TOL[dtype]


def _check_pooled(run, y, y2):
    """run(y or None, pooled, argmax): a bf16 convolution with its pool, un-pooled result kept or not; y: what the
    convolution alone gives.  Pooled values and positions bit for bit those of the separate pool, nothing written past
    them, and positions at an address that is a multiple of nothing (they are bytes)."""
    N, H, W, Cout = y.shape
    n = N * (H // 2) * (W // 2) * Cout
    po_chk = torch.empty((N, H // 2, W // 2, Cout), dtype=y.dtype, device="cuda")
    arg_chk = torch.empty((N, H // 2, W // 2, Cout), dtype=torch.uint8, device="cuda")
    B.vgg_maxpool2x2(B.BF16, N, H, W, Cout, y, po_chk, arg_chk)
    for keep, shift in ((True, 0), (False, 3)):
        po = torch.full((n + 1024,), -7.0, dtype=y.dtype, device="cuda")
        arg = torch.full((n + 1024,), 9, dtype=torch.uint8, device="cuda")
        run(y2 if keep else None, po, arg[shift:])
        torch.cuda.synchronize()
        if keep:
            assert torch.equal(y2.view(torch.int16), y.view(torch.int16))
        assert torch.equal(po[:n].view(torch.int16), po_chk.view(torch.int16).flatten())
        assert torch.equal(arg[shift:shift + n], arg_chk.flatten())
        assert (po[n:] == -7.0).all() and (arg[shift + n:] == 9).all() and (arg[:shift] == 9).all()


def _internal_conv():
    """The launcher behind the convolution entry points: the whole passes call it with pools that the public entry
    point does not take (images that 16-pixel patches do not divide, on the kernel for launches of few tiles)."""
    out = subprocess.run(["nm", "-D", "--defined-only", B.LIB_PATH], capture_output=True, text=True, check=True).stdout
    names = [w for line in out.splitlines() for w in line.split()[-1:] if w.startswith("_ZN3vgg13conv3x3_igemmE")]
    assert len(names) == 1, names
    f = B.lib()[names[0]]
    v, i = ctypes.c_void_p, ctypes.c_int
    f.argtypes, f.restype = [i] * 6 + [v] * 7 + [i, v, ctypes.c_size_t, v], i
    return f


@pytest.mark.parametrize("shape", [(1, 14, 14, 512, 512), (3, 14, 14, 512, 512), (1, 28, 28, 512, 512), (1, 56, 56, 256, 256), (2, 30, 44, 256, 40),
                                   (1, 20, 30, 416, 72), (2, 12, 100, 512, 64)])
def test_conv3x3_bf16_small_launches_with_their_pool(shape):
    """The pool that whole passes at small batches take in the kernel for launches of few tiles, patches sticking out of the
    image on both sides: against the same convolution without it and the separate pool, bit for bit."""
    dtype = B.BF16
    N, H, W, Cin, Cout = shape
    assert B.vgg_conv3x3_plan(B.PLAN_FWD, dtype, N, H, W, Cin, Cout)[0] in (12, 13)
    d = synth.conv_layer_inputs(N, H, W, Cin, Cout, seed=sum(shape) + 3)
    x, wp, b = to_nhwc(d["x"], dtype), _pack(dtype, d["w"]), dev(d["b"])
    y = torch.empty((N, H, W, Cout), dtype=TDT[dtype], device="cuda")
    B.vgg_conv3x3_fwd(dtype, N, H, W, Cin, Cout, x, wp, b, y, 1, ws_bytes(B.vgg_conv3x3_fwd_workspace_bytes(dtype, N, H, W, Cin, Cout)))
    conv, stream = _internal_conv(), torch.cuda.current_stream().cuda_stream

    def run(yy, po, arg):
        assert conv(dtype, N, H, W, Cin, Cout, x.data_ptr(), wp.data_ptr(), b.data_ptr(), None, yy.data_ptr() if yy is not None else None,
                    po.data_ptr(), arg.data_ptr(), 1, None, 0, stream) == 0

    _check_pooled(run, y, torch.empty_like(y))


@pytest.mark.parametrize("shape,kernel", [
    ((1, 14, 14, 512, 512), 13),    # eight waves, two chunks each; consecutive pixels that end inside a tile
    ((2, 30, 44, 256, 36), 12),     # two chunks per wave; patches that stick out on both sides; a ragged channel tile
    ((5, 16, 48, 288, 100), 12),    # nine chunks in three ranges; patches that divide the image
    ((1, 56, 56, 416, 64), 13),     # thirteen chunks in five ranges, the last one short
    ((10, 14, 14, 512, 512), 12),   # eight ranges for four waves (496 tiles)
    ((3, 30, 70, 96, 132), 9),      # an image row longer than the halo of 256 pixels
    ((12, 7, 9, 544, 260), 13),     # seventeen chunks in six ranges for eight waves; tiles that cross images
    ((4, 28, 28, 256, 516), 8),     # 128-pixel tiles, the sums folded over four ranges; a ragged channel tile
    ((2, 56, 56, 256, 256), 9),     # ... with the larger halo
    ((41, 14, 14, 384, 512), 10),   # 128-pixel tiles, nine taps of weights ahead (252 tiles)
    ((9, 30, 57, 384, 200), 11),    # ... with the larger halo
    ((9, 24, 16, 96, 512), 8),      # 128-pixel patches
    ((6, 30, 57, 96, 200), 9),      # 128 consecutive pixels, the larger halo, a ragged channel tile
    ((9, 32, 16, 96, 520), 8),      # 128-pixel patches whose pool can be fused, a ragged channel tile
    ((5, 32, 32, 384, 512), 10),    # ... with nine taps of weights ahead
])
def test_conv3x3_bf16_small_and_medium_launches(shape, kernel):
    """The kernels that launches of few tiles take, at the edges of their tiles and splits: forward and masked data
    gradient (of the layer with the channel counts exchanged) against the oracle, element by element, nothing
    written past the tensors; fused pool against the separate one where the sizes allow it."""
    dtype = B.BF16
    N, H, W, Cin, Cout = shape
    assert B.vgg_conv3x3_plan(B.PLAN_FWD, dtype, N, H, W, Cin, Cout)[0] == kernel
    d = synth.conv_layer_inputs(N, H, W, Cin, Cout, seed=sum(shape))
    x, n = to_nhwc(d["x"], dtype), N * H * W * Cout
    wp = _pack(dtype, d["w"])
    buf = torch.full((n + 4096,), -7.0, dtype=TDT[dtype], device="cuda")
    y = buf[:n].view(N, H, W, Cout)
    ws = ws_bytes(B.vgg_conv3x3_fwd_workspace_bytes(dtype, N, H, W, Cin, Cout))
    B.vgg_conv3x3_fwd(dtype, N, H, W, Cin, Cout, x, wp, dev(d["b"]), y, 1, ws)
    torch.cuda.synchronize()
    assert max_rel_err(from_nhwc(y), R.conv3x3_fwd(d["x"], d["w"], d["b"], relu=True)) <= TOL[dtype]
    assert (buf[n:] == -7.0).all()
    if H % 16 == 0 and W % 16 == 0 and Cout % 8 == 0:
        assert B.vgg_conv3x3_plan(B.PLAN_FWD_POOL, dtype, N, H, W, Cin, Cout)[0] == kernel
        y2 = torch.empty_like(y)
        _check_pooled(lambda yy, po, arg: B.vgg_conv3x3_fwd_pool(dtype, N, H, W, Cin, Cout, x, wp, dev(d["b"]), yy, po, 1, ws,
                                                                 argmax=arg), y, y2)
    d = synth.conv_layer_inputs(N, H, W, Cout, Cin, seed=sum(shape) + 1)
    assert B.vgg_conv3x3_plan(B.PLAN_BWD_DATA, dtype, N, H, W, Cout, Cin)[0] == kernel
    xs = to_nhwc(d["x"], dtype)
    ws = ws_bytes(B.vgg_conv3x3_bwd_data_workspace_bytes(dtype, N, H, W, Cout, Cin))
    buf.fill_(-7.0)
    B.vgg_conv3x3_bwd_data(dtype, N, H, W, Cout, Cin, to_nhwc(d["dy"], dtype), _pack(dtype, d["w"], flip=1), xs, y, ws)
    torch.cuda.synchronize()
    assert max_rel_err(from_nhwc(y), R.conv3x3_bwd_data(d["dy"], d["w"]) * (from_nhwc(xs) > 0)) <= TOL[dtype]
    assert (buf[n:] == -7.0).all()


@pytest.mark.parametrize("shape,kernel,columns", [
    ((1, 7, 9, 512, 20), 13, 16),       # a last column of four channels; one workgroup walks past the only tile's pixels
    ((1, 16, 16, 256, 68), 12, 16),     # four waves; patches, a last column of four channels
    ((1, 32, 16, 320, 140), 13, 16),    # five ranges for eight waves
    ((1, 21, 58, 256, 36), 12, 16),     # patches that stick out of the image
    ((1, 16, 64, 512, 252), 13, 16),    # 128 tiles of 32 channels, the last launch with columns of sixteen
    ((1, 16, 64, 512, 260), 13, 32),    # ... and the first with columns of 32
])
def test_conv3x3_bf16_sixteen_channel_columns(shape, kernel, columns):
    """Launches for at most half the CUs take columns of sixteen channels: as the other small launches, against the oracle."""
    N, H, W, Cin, Cout = shape
    assert B.vgg_conv3x3_plan(B.PLAN_FWD, B.BF16, N, H, W, Cin, Cout)[2] == columns
    test_conv3x3_bf16_small_and_medium_launches(shape, kernel)


@pytest.mark.parametrize("shape,kernel", [
    ((1, 5, 9, 64, 20), 1),        # two chunks, part of one tile, a last column of four channels
    ((3, 15, 8, 192, 144), 8),     # six chunks; tiles that cross images
    ((1, 32, 48, 160, 72), 8),     # five chunks; patches that divide the image: pool
    ((2, 30, 44, 96, 200), 9),     # a last column of 72 channels
    ((8, 32, 32, 96, 128), 8),     # 64 tiles; pool
    ((8, 32, 32, 96, 132), 8),     # a last column of four channels
    ((6, 13, 26, 224, 260), 8),    # seven chunks
])
def test_conv3x3_bf16_short_contractions_on_few_tiles(shape, kernel):
    """Contractions of two to seven chunks on a few workgroups, which no kernel splits (forward passes and training share the
    order of their sums): against the oracle, element by element, and the fused pool against the separate one, bit for bit."""
    dtype = B.BF16
    N, H, W, Cin, Cout = shape
    info = B.vgg_conv3x3_plan(B.PLAN_FWD, dtype, N, H, W, Cin, Cout)
    assert info[0] == kernel and info[5] == 1
    d = synth.conv_layer_inputs(N, H, W, Cin, Cout, seed=sum(shape))
    x, wp, b, n = to_nhwc(d["x"], dtype), _pack(dtype, d["w"]), dev(d["b"]), N * H * W * Cout
    ws = ws_bytes(B.vgg_conv3x3_fwd_workspace_bytes(dtype, N, H, W, Cin, Cout))
    buf = torch.full((n + 4096,), -7.0, dtype=TDT[dtype], device="cuda")
    y = buf[:n].view(N, H, W, Cout)
    B.vgg_conv3x3_fwd(dtype, N, H, W, Cin, Cout, x, wp, b, y, 1, ws)
    torch.cuda.synchronize()
    assert max_rel_err(from_nhwc(y), R.conv3x3_fwd(d["x"], d["w"], d["b"], relu=True)) <= TOL[dtype]
    assert (buf[n:] == -7.0).all()
    if H % 16 == 0 and W % 16 == 0 and Cout % 8 == 0:
        po = torch.full((n // 4 + 1024,), -7.0, dtype=TDT[dtype], device="cuda")
        B.vgg_conv3x3_fwd_pool(dtype, N, H, W, Cin, Cout, x, wp, b, None, po, 1, ws)
        chk = torch.empty((N, H // 2, W // 2, Cout), dtype=TDT[dtype], device="cuda")
        B.vgg_maxpool2x2(dtype, N, H, W, Cout, y, chk)
        torch.cuda.synchronize()
        assert torch.equal(po[:n // 4].view(torch.int16), chk.view(torch.int16).flatten()) and (po[n // 4:] == -7.0).all()


@pytest.mark.parametrize("shape,kernel", [
    ((7, 45, 60, 96, 200), 17),         # three chunks; a last tile of 84 pixels, a last column of 72 channels
    ((19, 36, 32, 128, 134), 17),       # patches of 12 x 16; a channel count that 16-byte stores do not divide
    ((30, 24, 13, 416, 460), 18),       # thirteen chunks, nine taps of weights ahead; tiles that cross images
    ((14, 41, 23, 128, 264), 17),       # a last column of eight channels
])
def test_conv3x3_bf16_192_pixel_tiles(shape, kernel):
    """192-pixel tiles at their edges: as the other medium launches, against the oracle."""
    test_conv3x3_bf16_small_and_medium_launches(shape, kernel)


@pytest.mark.parametrize("shape,kernel", [((1, 160, 100, 70400, 8), 12), ((83, 14, 14, 70400, 8), 13)])
def test_conv3x3_bf16_small_launches_of_large_inputs(shape, kernel):
    """Few tiles of an input beyond 2 GiB (patches; consecutive pixels), whose offsets count from a tile's halo: images' corners and
    edges and pixels behind the first 2 GiB against float64, zeros around the images included."""
    N, H, W, Cin, Cout = shape
    assert N * H * W * Cin * 2 > 2 ** 31 and B.vgg_conv3x3_plan(B.PLAN_FWD, B.BF16, N, H, W, Cin, Cout)[0] == kernel
    g = torch.Generator(device="cuda").manual_seed(Cin)
    x = torch.empty((N, H, W, Cin), dtype=torch.bfloat16, device="cuda").normal_(generator=g)
    w = (torch.randn((Cout, Cin, 3, 3), generator=g, device="cuda") / (9 * Cin) ** 0.5).bfloat16().float()
    wp = torch.empty((9 * Cout * B.vgg_padded_channels(B.BF16, Cin),), dtype=torch.bfloat16, device="cuda")
    B.vgg_conv_pack_weights(B.BF16, Cin, Cout, w, wp, 0)
    y = torch.empty((N, H, W, Cout), dtype=torch.bfloat16, device="cuda")
    B.vgg_conv3x3_fwd(B.BF16, N, H, W, Cin, Cout, x, wp, None, y, 0, ws_bytes(B.vgg_conv3x3_fwd_workspace_bytes(B.BF16, N, H, W, Cin, Cout)))
    torch.cuda.synchronize()
    past = 2 ** 31 // (2 * Cin)                               # the pixel that 2 GiB end in
    w64 = w.double()
    for m in {0, W - 1, H * W - 1, (N - 1) * H * W, past - 1, past, past + 1, past + W, N * H * W - W, N * H * W - 1}:
        n, h, v = m // (H * W), m // W % H, m % W
        want = torch.zeros((Cout,), dtype=torch.float64, device="cuda")
        for t in range(9):
            hh, vv = h + t // 3 - 1, v + t % 3 - 1
            if 0 <= hh < H and 0 <= vv < W:
                want += w64[:, :, t // 3, t % 3] @ x[n, hh, vv].double()
        assert (y[n, h, v].double() - want).abs().max().item() <= 2.0 ** -7 * 4, m   # (results of N(0,1): below 4; half an ulp of bf16 is 2^-9 of them)


@pytest.mark.parametrize("shape", [(1, 14, 14, 576, 512), (2, 7, 9, 1024, 200), (3, 20, 19, 768, 132), (2, 12, 36, 576, 72)])
def test_conv3x3_bf16_split_over_workgroups(shape):
    """More ranges than the waves of one workgroup share (more than 512 input channels): the ranges go to workgroups of
    their own again.  Forward and masked data gradient against the oracle; without a workspace the call is refused."""
    dtype = B.BF16
    N, H, W, Cin, Cout = shape
    plan = B.vgg_conv3x3_plan(B.PLAN_FWD, dtype, N, H, W, Cin, Cout)
    assert plan[0] in (1, 2) and plan[5] > 8 and plan[6] == plan[4] * -(-Cout // 64) * plan[5]
    d = synth.conv_layer_inputs(N, H, W, Cin, Cout, seed=sum(shape))
    x = to_nhwc(d["x"], dtype)
    y = torch.empty((N, H, W, Cout), dtype=TDT[dtype], device="cuda")
    ws = ws_bytes(B.vgg_conv3x3_fwd_workspace_bytes(dtype, N, H, W, Cin, Cout))
    B.vgg_conv3x3_fwd(dtype, N, H, W, Cin, Cout, x, _pack(dtype, d["w"]), dev(d["b"]), y, 1, ws)
    torch.cuda.synchronize()
    assert max_rel_err(from_nhwc(y), R.conv3x3_fwd(d["x"], d["w"], d["b"], relu=True)) <= TOL[dtype]
    with pytest.raises(B.VggError):
        B.vgg_conv3x3_fwd(dtype, N, H, W, Cin, Cout, x, _pack(dtype, d["w"]), dev(d["b"]), y, 1, None)
    d = synth.conv_layer_inputs(N, H, W, Cout, Cin, seed=sum(shape) + 1)
    assert B.vgg_conv3x3_plan(B.PLAN_BWD_DATA, dtype, N, H, W, Cout, Cin) == plan
    xs = to_nhwc(d["x"], dtype)
    ws = ws_bytes(B.vgg_conv3x3_bwd_data_workspace_bytes(dtype, N, H, W, Cout, Cin))
    B.vgg_conv3x3_bwd_data(dtype, N, H, W, Cout, Cin, to_nhwc(d["dy"], dtype), _pack(dtype, d["w"], flip=1), xs, y, ws)
    torch.cuda.synchronize()
    assert max_rel_err(from_nhwc(y), R.conv3x3_bwd_data(d["dy"], d["w"]) * (from_nhwc(xs) > 0)) <= TOL[dtype]


@pytest.mark.parametrize("shape,kernel,bn", [
    ((1, 9, 9, 48, 40), 16, 64), ((4, 64, 64, 32, 64), 14, 64), ((3, 20, 21, 40, 130), 16, 64), ((12, 40, 41, 16, 24), 15, 64),
    # split over workgroups, whole and half last chunks; patches of wide images
    ((1, 12, 40, 80, 72), 16, 64), ((2, 43, 54, 136, 72), 15, 64), ((9, 28, 28, 208, 64), 16, 64), ((20, 28, 28, 112, 132), 14, 64), ((3, 24, 95, 72, 112), 16, 64), ((5, 65, 83, 32, 100), 16, 64), ((33, 64, 64, 32, 72), 14, 128),
    ((5, 56, 56, 16, 132), 15, 64), ((43, 56, 56, 32, 132), 15, 128), ((43, 56, 56, 40, 128), 15, 128), ((50, 14, 14, 80, 512), 16, 64), ((100, 13, 14, 32, 268), 16, 64)])
def test_conv3x3_fp32_in_three_parts(shape, kernel, bn):
    """The fp32 kernels on the bf16 matrix unit: half a last chunk, ragged channels, every tile, pooled and masked.  Sums of at
    most 720 products, of each of which at most 2^-24 is left out, in fp32: 2e-6 of the largest output against the oracle."""
    N, H, W, Cin, Cout = shape
    plan = B.vgg_conv3x3_plan(B.PLAN_FWD, B.F32, N, H, W, Cin, Cout)
    assert plan[0] == kernel and plan[2] == bn, plan
    d = synth.conv_layer_inputs(N, H, W, Cin, Cout, seed=sum(shape))
    n = N * H * W * Cout
    y = torch.full((n + 256,), -7.0, device="cuda")
    ws = ws_bytes(B.vgg_conv3x3_fwd_workspace_bytes(B.F32, N, H, W, Cin, Cout))
    x, w = to_nhwc(d["x"], B.F32), _pack(B.F32, d["w"])
    B.vgg_conv3x3_fwd(B.F32, N, H, W, Cin, Cout, x, w, dev(d["b"]), y, 1, ws)
    torch.cuda.synchronize()
    got = y[:n].view(N, H, W, Cout)
    assert max_rel_err(from_nhwc(got), R.conv3x3_fwd(d["x"], d["w"], d["b"], relu=True)) <= 2e-6
    assert (y[n:] == -7.0).all()
    if H % 16 == 0 and W % 16 == 0 and Cout % 4 == 0:
        po, arg = torch.empty((N, H // 2, W // 2, Cout), device="cuda"), torch.empty((N, H // 2, W // 2, Cout), dtype=torch.uint8, device="cuda")
        B.vgg_conv3x3_fwd_pool(B.F32, N, H, W, Cin, Cout, x, w, dev(d["b"]), None, po, 1, ws=ws, argmax=arg)
        pref, aref = R.maxpool2x2(from_nhwc(got))
        assert np.array_equal(from_nhwc(po), pref) and np.array_equal(arg.permute(0, 3, 1, 2).cpu().numpy(), aref)
    if Cin % 16 == 0:                                         # data gradient of the mirrored layer
        xs = torch.randn((N, H, W, Cout), device="cuda")
        B.vgg_conv3x3_bwd_data(B.F32, N, H, W, Cout, Cin, x, w, xs, y, ws_bytes(B.vgg_conv3x3_bwd_data_workspace_bytes(B.F32, N, H, W, Cout, Cin)))
        torch.cuda.synchronize()
        ref = R.conv3x3_fwd(d["x"], d["w"], None, relu=False) * (from_nhwc(xs) > 0)
        assert max_rel_err(from_nhwc(y[:n].view(N, H, W, Cout)), ref) <= 2e-6


def test_conv3x3_fp32_in_three_parts_infinities_and_range():
    """Infinities, NaN, overflow and values near both ends of the range come out as in fp32 arithmetic."""
    N, H, W, Cin, Cout = 1, 16, 32, 32, 64
    assert B.vgg_conv3x3_plan(B.PLAN_FWD, B.F32, N, H, W, Cin, Cout)[0] in (14, 15, 16)
    rng = np.random.default_rng(5)
    x, w = rng.standard_normal((N, Cin, H, W)).astype(np.float32), rng.standard_normal((Cout, Cin, 3, 3)).astype(np.float32)
    w[:8] = 1.0                                               # second and third parts are zero
    w[8:12] = 0.0                                             # infinity times zero
    x[0, 3, 2, 4], x[0, 5, 9, 20], x[0, 7, 9, 21], x[0, 9, 14, 9], x[0, 1, 5, 28] = np.inf, np.inf, -np.inf, np.nan, 3.2e38
    y = torch.empty((N, H, W, Cout), device="cuda")
    ws = ws_bytes(B.vgg_conv3x3_fwd_workspace_bytes(B.F32, N, H, W, Cin, Cout))
    B.vgg_conv3x3_fwd(B.F32, N, H, W, Cin, Cout, to_nhwc(x, B.F32), _pack(B.F32, w), None, y, 0, ws)
    torch.cuda.synchronize()
    got = from_nhwc(y)
    with np.errstate(all="ignore"):
        ref = torch.nn.functional.conv2d(torch.from_numpy(x).double(), torch.from_numpy(w).double(), padding=1).float().numpy()
    ok = ~np.isnan(ref)                                       # (a tile leaves through a maximum, which drops NaN for -infinity)
    assert np.array_equal(np.isfinite(got), np.isfinite(ref)) and np.isposinf(ref).any() and (~ok).any()
    for f in (np.isposinf, np.isneginf):
        assert np.array_equal(f(got[ok]), f(ref[ok]))
    for s in (2.0 ** -90, 2.0 ** 100):
        xs = (rng.standard_normal((N, Cin, H, W)) * s).astype(np.float32)
        B.vgg_conv3x3_fwd(B.F32, N, H, W, Cin, Cout, to_nhwc(xs, B.F32), _pack(B.F32, w), None, y, 0, ws)
        torch.cuda.synchronize()
        assert max_rel_err(from_nhwc(y), R.conv3x3_fwd(xs, w, None, relu=False)) <= 2e-6


def da_partial_sum_bytes(N, In, Out):
    """Workspace of da's partial sums in the fp32 dense backward: 512 workgroups rounded up to whole splits of the tiles of 128 rows x
    256 inputs, at least 64 outputs each."""
    tiles = -(-In // 256) * -(-N // 128)
    splits = max(1, min(-(-512 // tiles), -(-Out // 64)))
    per_split = -(-(-(-Out // splits)) // 16) * 16
    return -(-(-(-Out // per_split) * N * In * 4) // 256) * 256


def dz_in_parts(N, In, Out):
    """Whether the fp32 dense backward asks for room for dz in parts (two copies, 3 KB per 32 outputs and sixteen rows) as well."""
    parts = B.vgg_fc_bwd_workspace_bytes(B.F32, N, In, Out) - da_partial_sum_bytes(N, In, Out)
    assert parts in (0, 2 * -(-Out // 32) * -(-N // 16) * 3072)
    return parts > 0


def _full_mantissas(shape, seed):
    """fp32 values in [1, 2) with random 24-bit significands, among them 0x3f80ffff, of which a truncating split into 8-bit
    parts leaves out the most."""
    g = torch.Generator().manual_seed(seed)
    v = torch.randint(0, 1 << 23, shape, generator=g, dtype=torch.int32) | 0x3f800000
    v.view(-1)[::7] = 0x3f80ffff
    return v.view(torch.float32).cuda()


def _three_part_call(op, lone, N=64, parts=True):
    """(result, the same in 64 bits) of an fp32 call on the bf16 matrix unit, all operands positive; lone: one product per result.
    Dense backward: N rows; parts: whether the workspace has room for dz in parts."""
    if op in ("dw", "da"):
        In, Out = (640, 512) if op == "dw" else (512, 4096) if parts and N <= 128 else (1032, 4096)
        assert dz_in_parts(N, In, Out) == (N <= 128 and (op == "dw" or In == 512))
        a, w, dz = _full_mantissas((N, In), 1), _full_mantissas((Out, In), 2), _full_mantissas((N, Out), 3)
        if lone:
            keep = torch.zeros_like(dz)
            keep[3 if op == "dw" else slice(None), slice(None) if op == "dw" else 7] = 1.0
            dz = dz * keep
        dw, db, da = torch.empty((Out, In), device="cuda"), torch.empty((Out,), device="cuda"), torch.empty((N, In), device="cuda")
        size = B.vgg_fc_bwd_workspace_bytes(B.F32, N, In, Out) if parts else da_partial_sum_bytes(N, In, Out)
        B.vgg_fc_bwd(B.F32, N, In, Out, a, w, dz, dw, db, da, 0, ws_bytes(size))
        torch.cuda.synchronize()
        return (dw, dz.double().t() @ a.double()) if op == "dw" else (da, dz.double() @ w.double())
    N, H, W, Cin, Cout = (3, 28, 28, 512, 128) if op != "wgrad" else (9, 28, 28, 96, 128)
    plan = B.vgg_conv3x3_plan({"fwd": B.PLAN_FWD, "bwd_data": B.PLAN_BWD_DATA, "wgrad": B.PLAN_BWD_WEIGHT}[op], B.F32, N, H, W,
                              *((Cout, Cin) if op == "bwd_data" else (Cin, Cout)))
    assert plan[0] in ((114,) if op == "wgrad" else (14, 15, 16)), plan
    x, g = _full_mantissas((N, H, W, Cin), 4), _full_mantissas((N, H, W, Cout), 5)
    pad = lambda t: torch.nn.functional.pad(t.double(), (0, 0, 1, 1, 1, 1))
    if op == "wgrad":
        if lone:
            keep = torch.zeros_like(g)
            keep[1, 9, 13] = 1.0
            g = g * keep
        dw, db = torch.empty((9, Cout, Cin), device="cuda"), torch.empty((Cout,), device="cuda")
        B.vgg_conv3x3_bwd_weight(B.F32, N, H, W, Cin, Cout, x, g, dw, db, ws_bytes(B.vgg_conv3x3_bwd_weight_workspace_bytes(B.F32, N, H, W, Cin, Cout)))
        torch.cuda.synchronize()
        xp, g2 = pad(x), g.double().reshape(-1, Cout).t()
        return dw, torch.stack([g2 @ xp[:, t // 3:t // 3 + H, t % 3:t % 3 + W].reshape(-1, Cin) for t in range(9)])
    if lone:                                                  # one pixel of nine, one channel: every output meets one of them
        keep = torch.zeros_like(x)
        keep[:, 1::3, 1::3, 5] = 1.0
        x = x * keep
    w = _full_mantissas((9, Cout, Cin), 6)                    # (packed: Cin is a multiple of 16)
    y = torch.empty((N, H, W, Cout), device="cuda")
    if op == "fwd":
        B.vgg_conv3x3_fwd(B.F32, N, H, W, Cin, Cout, x, w, None, y, 0, ws_bytes(B.vgg_conv3x3_fwd_workspace_bytes(B.F32, N, H, W, Cin, Cout)))
    else:
        B.vgg_conv3x3_bwd_data(B.F32, N, H, W, Cout, Cin, x, w, None, y, ws_bytes(B.vgg_conv3x3_bwd_data_workspace_bytes(B.F32, N, H, W, Cout, Cin)))
    torch.cuda.synchronize()
    xp = pad(x)
    ref = sum(xp[:, t // 3:t // 3 + H, t % 3:t % 3 + W].reshape(-1, Cin) @ w[t].double().t() for t in range(9)).view(N, H, W, Cout)
    return y[:, :27, :27], ref[:, :27, :27]                   # (lone: pixel 25 is the last kept one, row and column 27 meet none)


@pytest.mark.parametrize("lone", [True, False])
@pytest.mark.parametrize("op", ["fwd", "bwd_data", "wgrad", "dw", "da"])
def test_fp32_products_in_three_parts_without_a_bias(op, lone, N=64, parts=True):
    """Every kernel that multiplies fp32 in three parts, positive operands with full significands.  One product: at most 2^-24 of
    it is left out and the result rounded (2^-24).  Sums of 64 to 7056 products: no element off by more than 5e-6 (a sum's own
    rounding), and in both no bias: a mean signed error of 1e-8, where rounding to nearest gives 1e-9 over as many results."""
    got, ref = _three_part_call(op, lone, N, parts)
    err = (got.double() - ref) / ref
    assert err.abs().max().item() <= (2.0 ** -23 if lone else 5e-6)
    assert abs(err.mean().item()) <= 1e-8


# Dense backward kernels that split dz themselves: workspaces without room for its parts (three to eight blocks of sixteen rows), and more than
# 128 rows (blocks of two and three row tiles).
SPLIT_DZ_ROWS = [(64, False), (80, False), (128, False), (200, True), (257, True)]


@pytest.mark.parametrize("lone", [True, False])
@pytest.mark.parametrize("N,parts", SPLIT_DZ_ROWS)
@pytest.mark.parametrize("op", ["dw", "da"])
def test_fp32_dense_products_in_three_parts_without_a_bias(op, N, parts, lone):
    """The same, for the dense backward kernels that split dz themselves."""
    test_fp32_products_in_three_parts_without_a_bias(op, lone, N, parts)


@pytest.mark.parametrize("N,parts", [(48, False)] + SPLIT_DZ_ROWS)
def test_fp32_dense_backward_in_three_parts_keeps_nan_and_the_largest_values(N, parts):
    """A NaN whose payload lies below the first part stays one; values that round to infinity in bf16 stay finite; infinities
    as in fp32 arithmetic: both products, and dW where da is not asked for."""
    In, Out = 136, 64
    g = torch.Generator().manual_seed(8)
    a, w, dz = (torch.randn(s, generator=g) for s in ((N, In), (Out, In), (N, Out)))
    nan, largest = torch.tensor([0x7f800001, -0x7ffffe], dtype=torch.int32).view(torch.float32), torch.finfo(torch.float32).max
    a[5, 7], w[2, 9], a[6, 70], w[33, 100], a[9, 11] = nan[0], nan[1], float("inf"), float("-inf"), largest
    dz[9], dz[:, 40] = 0.25 * torch.sign(dz[9]), 0.0
    w[40, 50] = -largest
    dz[12, 40] = 0.5
    dw, da, alone = torch.empty((Out, In), device="cuda"), torch.empty((N, In), device="cuda"), torch.empty((Out, In), device="cuda")
    assert dz_in_parts(N, In, Out) == (N <= 128)
    size = B.vgg_fc_bwd_workspace_bytes(B.F32, N, In, Out) if parts else da_partial_sum_bytes(N, In, Out)
    B.vgg_fc_bwd(B.F32, N, In, Out, a.cuda(), w.cuda(), dz.cuda(), dw, None, da, 0, ws_bytes(size))
    B.vgg_fc_bwd(B.F32, N, In, Out, a.cuda(), w.cuda(), dz.cuda(), alone, None, None, 0, None)
    torch.cuda.synchronize()
    dw_ref, da_ref = dz.double().t() @ a.double(), dz.double() @ w.double()
    for got, ref in ((dw.cpu(), dw_ref), (alone.cpu(), dw_ref), (da.cpu(), da_ref)):
        assert torch.equal(got.isnan(), ref.isnan()) and ref.isnan().any()
        assert torch.equal(got.isposinf(), ref.isposinf()) and torch.equal(got.isneginf(), ref.isneginf()) and ref.isinf().any()
        big = ref.isfinite() & (ref.abs() > 1e37)
        assert big.any() and ((got[big].double() - ref[big]) / ref[big]).abs().max() <= 2.0 ** -23


def test_fp32_in_three_parts_keeps_nan_and_the_largest_values():
    """As above, dense backward with dz in parts ahead of the products, and the weight gradient of a convolution.  (Their results pass
    through no maximum.)"""
    test_fp32_dense_backward_in_three_parts_keeps_nan_and_the_largest_values(48, True)
    nan = torch.tensor([0x7f800001, -0x7ffffe], dtype=torch.int32).view(torch.float32)
    g = torch.Generator().manual_seed(8)
    N, H, W, Cin, Cout = 3, 28, 28, 32, 64
    assert B.vgg_conv3x3_plan(B.PLAN_BWD_WEIGHT, B.F32, N, H, W, Cin, Cout)[0] == 114
    x, gr = torch.randn((N, H, W, Cin), generator=g), torch.randn((N, H, W, Cout), generator=g)
    x[0, 3, 4, 6], gr[1, 7, 8, 9] = nan[0], nan[1]
    dw, db = torch.empty((9, Cout, Cin), device="cuda"), torch.empty((Cout,), device="cuda")
    B.vgg_conv3x3_bwd_weight(B.F32, N, H, W, Cin, Cout, x.cuda(), gr.cuda(), dw, db, ws_bytes(B.vgg_conv3x3_bwd_weight_workspace_bytes(B.F32, N, H, W, Cin, Cout)))
    torch.cuda.synchronize()
    want = torch.zeros((9, Cout, Cin), dtype=torch.bool)
    want[:, :, 6], want[:, 9] = True, True
    assert torch.equal(dw.cpu().isnan(), want) and torch.equal(dw.cpu().isfinite(), ~want)


@pytest.mark.parametrize("dtype,shape,kernel", [
    (B.F32, (2, 46, 79, 32, 36), 1), (B.F32, (1, 24, 200, 96, 64), 1), (B.F32, (1, 97, 97, 48, 132), 1), (B.F32, (3, 63, 65, 3, 20), 1),
    (B.F32, (9, 66, 66, 16, 192), 0), (B.F32, (1, 6, 150, 16, 32), 0),
    (B.BF16, (2, 46, 79, 32, 36), 1), (B.BF16, (3, 62, 75, 64, 200), 1), (B.BF16, (4, 36, 100, 96, 256), 4), (B.BF16, (2, 36, 100, 160, 520), 4),
    (B.BF16, (1, 24, 200, 512, 64), 13), (B.BF16, (9, 66, 66, 32, 136), 0)])
def test_conv3x3_wide_images(dtype, shape, kernel):
    """Rows too long for the direct-to-LDS kernels' halo of consecutive pixels: patches that stick out of the image where that
    pays, else the staged kernel; no partial sums in memory, no scratch beyond the padded copy.  Forward against the
    oracle, nothing written past the tensor; data gradient of the mirrored layer with its mask."""
    N, H, W, Cin, Cout = shape
    plan = B.vgg_conv3x3_plan(B.PLAN_FWD, dtype, N, H, W, Cin, Cout)
    assert plan[0] == kernel and plan[3] == (kernel != 0) and (plan[5] == 1 or kernel == 13), plan
    cp, size = B.vgg_padded_channels(dtype, Cin), 4 if dtype == B.F32 else 2
    padded = 0 if cp == Cin else -(-N * H * W * cp * size // 256) * 256
    assert B.vgg_conv3x3_fwd_workspace_bytes(dtype, N, H, W, Cin, Cout) == padded
    d = synth.conv_layer_inputs(N, H, W, Cin, Cout, seed=sum(shape))
    n = N * H * W * Cout
    buf = torch.full((n + 4096,), -7.0, dtype=TDT[dtype], device="cuda")
    y = buf[:n].view(N, H, W, Cout)
    ws = ws_bytes(B.vgg_conv3x3_fwd_workspace_bytes(dtype, N, H, W, Cin, Cout))
    B.vgg_conv3x3_fwd(dtype, N, H, W, Cin, Cout, to_nhwc(d["x"], dtype), _pack(dtype, d["w"]), dev(d["b"]), y, 1, ws)
    torch.cuda.synchronize()
    assert max_rel_err(from_nhwc(y), R.conv3x3_fwd(d["x"], d["w"], d["b"], relu=True)) <= TOL[dtype]
    assert (buf[n:] == -7.0).all()
    d = synth.conv_layer_inputs(N, H, W, Cout, Cin, seed=sum(shape) + 1)
    xs = to_nhwc(d["x"], dtype)
    ws = ws_bytes(B.vgg_conv3x3_bwd_data_workspace_bytes(dtype, N, H, W, Cout, Cin))
    buf.fill_(-7.0)
    B.vgg_conv3x3_bwd_data(dtype, N, H, W, Cout, Cin, to_nhwc(d["dy"], dtype), _pack(dtype, d["w"], flip=1), xs, y, ws)
    torch.cuda.synchronize()
    assert max_rel_err(from_nhwc(y), R.conv3x3_bwd_data(d["dy"], d["w"]) * (from_nhwc(xs) > 0)) <= TOL[dtype]
    assert (buf[n:] == -7.0).all()


@pytest.mark.parametrize("shape", FULL_SIZE_LAYERS)
def test_conv3x3_bf16_full_size_on_sampled_pixels(shape):
    """Forward and data gradient at the benchmark's sizes, in the launch configuration it times; the oracle
    computes the sampled pixels one neighbourhood at a time (all channels of each)."""
    N, H, W, Cin, Cout, kernel_fwd, kernel_bwd = shape
    dtype = B.BF16
    plan = B.vgg_conv3x3_plan(B.PLAN_FWD, dtype, N, H, W, Cin, Cout)
    assert plan[0] == kernel_fwd, plan
    assert B.vgg_conv3x3_plan(B.PLAN_BWD_DATA, dtype, N, H, W, Cin, Cout)[0] == kernel_bwd
    d = synth.conv_layer_inputs(N, H, W, Cin, Cout, seed=sum(shape[:5]))
    n, h, w = _sample_pixels(N, H, W, plan[1], 400, seed=H + Cin)
    x = to_nhwc(d["x"], dtype)
    # forward (bias, ReLU): the centre of the oracle's output over each 3x3 neighbourhood
    y = torch.empty((N, H, W, Cout), dtype=TDT[dtype], device="cuda")
    ws = ws_bytes(B.vgg_conv3x3_fwd_workspace_bytes(dtype, N, H, W, Cin, Cout))
    B.vgg_conv3x3_fwd(dtype, N, H, W, Cin, Cout, x, _pack(dtype, d["w"]), dev(d["b"]), y, 1, ws)
    torch.cuda.synchronize()
    ref = R.conv3x3_fwd(_patches(d["x"], n, h, w), d["w"], d["b"], relu=True)[:, :, 1, 1]
    got = y[torch.from_numpy(n).cuda(), torch.from_numpy(h).cuda(), torch.from_numpy(w).cuda()].float().cpu().numpy()
    assert max_rel_err(got, ref) <= TOL[dtype]
    del y
    # data gradient, without and with the (x > 0) factor of the layer below
    g = to_nhwc(d["dy"], dtype)
    dx = torch.empty((N, H, W, Cin), dtype=TDT[dtype], device="cuda")
    ws = ws_bytes(B.vgg_conv3x3_bwd_data_workspace_bytes(dtype, N, H, W, Cin, Cout))
    wtf = _pack(dtype, d["w"], flip=1)
    ref = R.conv3x3_bwd_data(_patches(d["dy"], n, h, w), d["w"])[:, :, 1, 1]
    idx = (torch.from_numpy(n).cuda(), torch.from_numpy(h).cuda(), torch.from_numpy(w).cuda())
    B.vgg_conv3x3_bwd_data(dtype, N, H, W, Cin, Cout, g, wtf, None, dx, ws)
    torch.cuda.synchronize()
    assert max_rel_err(dx[idx].float().cpu().numpy(), ref) <= TOL[dtype]
    B.vgg_conv3x3_bwd_data(dtype, N, H, W, Cin, Cout, g, wtf, x, dx, ws)
    torch.cuda.synchronize()
    keep = x[idx].float().cpu().numpy() > 0
    assert max_rel_err(dx[idx].float().cpu().numpy(), ref * keep) <= TOL[dtype]


@pytest.mark.parametrize("dtype", [B.F32, B.BF16])
@pytest.mark.parametrize("shape", CONV_SHAPES)
def test_conv3x3_bwd_weight(dtype, shape):
    _check_bwd_weight(dtype, shape, seed=sum(shape) + 2)


def _check_bwd_weight(dtype, shape, seed):
    """fp32, or bf16 operands (x and g rounded to bf16, fp32 sums and fp32 result)."""
    N, H, W, Cin, Cout = shape
    d = synth.conv_layer_inputs(N, H, W, Cin, Cout, seed=seed)
    dw_ref, db_ref = R.conv3x3_bwd_weight(d["x"], d["dy"])
    x = to_nhwc(d["x"], dtype)
    g = to_nhwc(d["dy"], dtype)
    cp = B.vgg_padded_channels(dtype, Cin)
    dwp = torch.full((9, Cout, cp), float("nan"), device="cuda")
    db = torch.empty((Cout,), device="cuda")
    ws = ws_bytes(B.vgg_conv3x3_bwd_weight_workspace_bytes(dtype, N, H, W, Cin, Cout))
    if dtype == B.BF16 and Cout % 8:
        with pytest.raises(B.VggError):      # 16-byte channel segments of g
            B.vgg_conv3x3_bwd_weight(dtype, N, H, W, Cin, Cout, x, g, dwp, db, ws)
        return
    B.vgg_conv3x3_bwd_weight(dtype, N, H, W, Cin, Cout, x, g, dwp, db, ws)
    torch.cuda.synchronize()
    dw = dwp[:, :, :Cin].reshape(3, 3, Cout, Cin).permute(2, 3, 0, 1)    # [t][co][ci] -> [co][ci][kh][kw]
    assert max_rel_err(dw.cpu().numpy(), dw_ref) <= TOL[dtype]
    assert max_rel_err(db.cpu().numpy(), db_ref) <= TOL[dtype]
    assert (dwp[:, :, Cin:] == 0).all()     # padding channels get exact zeros
    if dtype == B.F32:
        dw2 = torch.empty((Cout, Cin, 3, 3), device="cuda")
        B.vgg_conv_unpack_weights(Cin, Cout, dwp, dw2)
        torch.cuda.synchronize()
        assert torch.equal(dw2, dw)
    # run-to-run reproducibility of the split reduction
    dwp2 = torch.empty_like(dwp)
    B.vgg_conv3x3_bwd_weight(dtype, N, H, W, Cin, Cout, x, g, dwp2, db, ws)
    torch.cuda.synchronize()
    assert torch.equal(dwp, dwp2)


@pytest.mark.parametrize("shape", [(2, 24, 40, 72, 64), (3, 21, 37, 40, 72), (2, 7, 7, 16, 40), (1, 56, 56, 24, 128), (5, 8, 6, 200, 136)])
def test_conv3x3_bwd_weight_bf16_on_8x8_patches(shape):
    """bf16 weight gradient at sizes that 8 x 8 patches cover with fewer than 4 x 16 ones: dividing the image and
    sticking out of it, with wide and narrow (at most 16 and 32) input channels, against the oracle."""
    N, H, W, Cin, Cout = shape
    assert B.vgg_conv3x3_plan(B.PLAN_BWD_WEIGHT, B.BF16, N, H, W, Cin, Cout)[4] == N * -(-H // 8) * -(-W // 8)
    _check_bwd_weight(B.BF16, shape, seed=sum(shape) + 5)


@pytest.mark.parametrize("dtype,shape,splits", [(B.F32, (1, 8, 8, 16, 4), (1, 1)), (B.F32, (2, 7, 9, 16, 24), (2, 15)),
                                                (B.F32, (3, 30, 17, 16, 28), (16, 127)), (B.F32, (30, 56, 56, 16, 24), (128, 999)),
                                                (B.BF16, (1, 8, 8, 16, 8), (1, 15)), (B.BF16, (3, 30, 17, 16, 24), (16, 127)),
                                                (B.BF16, (20, 40, 40, 16, 40), (128, 999))])
def test_conv3x3_bwd_weight_partial_sums(dtype, shape, splits):
    """Each form of the pass that adds the partial sums, by their number, with outputs that end inside a workgroup."""
    N, H, W, Cin, Cout = shape
    assert splits[0] <= B.vgg_conv3x3_plan(B.PLAN_BWD_WEIGHT, dtype, N, H, W, Cin, Cout)[5] <= splits[1]
    _check_bwd_weight(dtype, shape, seed=sum(shape) + 9)


@pytest.mark.parametrize("shape,kernel", [((12, 43, 19, 24, 72), 108), ((9, 18, 34, 33, 64), 108), ((70, 7, 7, 40, 132), 108), ((40, 14, 14, 96, 200), 114),
                                          ((1, 64, 80, 16, 4), 116), ((2, 16, 32, 64, 64), 116), ((65, 3, 7, 16, 36), 100)])
def test_conv3x3_bwd_weight_fp32_in_three_parts(shape, kernel):
    """The fp32 weight gradient on the bf16 matrix unit: every patch shape, sticking out at the right and bottom, ragged
    channels, one and several patches per workgroup.  Sums of at most 9288 products, each exact to 2^-24: 3e-6 of the largest
    value against the oracle (fp32 sums of that length: 1e-6)."""
    N, H, W, Cin, Cout = shape
    assert B.vgg_conv3x3_plan(B.PLAN_BWD_WEIGHT, B.F32, N, H, W, Cin, Cout)[0] == kernel
    _check_bwd_weight(B.F32, shape, seed=sum(shape) + 6)
    d = synth.conv_layer_inputs(N, H, W, Cin, Cout, seed=sum(shape) + 6)
    dw_ref, db_ref = R.conv3x3_bwd_weight(d["x"], d["dy"])
    cp = B.vgg_padded_channels(B.F32, Cin)
    dwp, db = torch.empty((9, Cout, cp), device="cuda"), torch.empty((Cout,), device="cuda")
    B.vgg_conv3x3_bwd_weight(B.F32, N, H, W, Cin, Cout, to_nhwc(d["x"], B.F32), to_nhwc(d["dy"], B.F32), dwp, db,
                             ws_bytes(B.vgg_conv3x3_bwd_weight_workspace_bytes(B.F32, N, H, W, Cin, Cout)))
    torch.cuda.synchronize()
    dw = dwp[:, :, :Cin].reshape(3, 3, Cout, Cin).permute(2, 3, 0, 1)
    assert max_rel_err(dw.cpu().numpy(), dw_ref) <= 3e-6 and max_rel_err(db.cpu().numpy(), db_ref) <= 3e-6


@pytest.mark.parametrize("shape,kernel", [((3, 28, 28, 32, 64), 114), ((1, 56, 56, 40, 72), 114), ((3, 50, 66, 40, 72), 114), ((1, 45, 60, 96, 36), 116),
                                          ((2, 16, 32, 64, 64), 116), ((12, 43, 19, 24, 72), 108), ((70, 7, 7, 40, 132), 108)])
def test_conv3x3_bwd_weight_fp32_in_three_parts_infinities(shape, kernel):
    """An infinite or NaN x meets the pixels of g that the image has and no other: beside the columns and rows that a patch
    multiplies beyond its own or the image's last ones, a tap's sum is infinite, NaN or finite as in 64 bits."""
    N, H, W, Cin, Cout = shape
    assert B.vgg_conv3x3_plan(B.PLAN_BWD_WEIGHT, B.F32, N, H, W, Cin, Cout)[0] == kernel
    gen = torch.Generator().manual_seed(sum(shape))
    x, g = torch.randn((N, H, W, Cin), generator=gen), torch.randn((N, H, W, Cout), generator=gen)
    for c, (h, w, v) in enumerate([(3, W - 1, 1), (H - 1, 5, -1), (H - 1, W - 1, 1), (3, min(14, W - 2), 1), (2, min(15, W - 1), -1), (H - 1, 0, 1), (0, W - 1, 1),
                                   (min(7, H - 1), 6, 1), (min(8, H - 2), min(8, W - 2), 1)]):
        x[N - 1, h, w, c] = v * float("inf")
    x[0, 1, W - 1, 9] = float("nan")
    dw, db = torch.empty((9, Cout, B.vgg_padded_channels(B.F32, Cin)), device="cuda"), torch.empty((Cout,), device="cuda")
    B.vgg_conv3x3_bwd_weight(B.F32, N, H, W, Cin, Cout, x.cuda(), g.cuda(), dw, db, ws_bytes(B.vgg_conv3x3_bwd_weight_workspace_bytes(B.F32, N, H, W, Cin, Cout)))
    torch.cuda.synchronize()
    xp, g2 = torch.nn.functional.pad(x.double(), (0, 0, 1, 1, 1, 1)), g.double().reshape(-1, Cout).t().contiguous()
    ref = torch.stack([g2 @ xp[:, t // 3:t // 3 + H, t % 3:t % 3 + W].reshape(-1, Cin) for t in range(9)])
    got = dw[:, :, :Cin].cpu()
    for f in (torch.isnan, torch.isposinf, torch.isneginf):
        assert torch.equal(f(got), f(ref))
    ok = ref.isfinite()
    assert ok[:, :, 0].any() and not ok[:, :, 0].all()        # (the last column's infinity: not in the taps that look left of it)
    assert (got[ok].double() - ref[ok]).abs().max() <= 3e-6 * ref[ok].abs().max()


@pytest.mark.parametrize("shape,kernel", [((3, 50, 66, 40, 72), 114), ((3, 8, 100, 16, 64), 116), ((1, 45, 60, 96, 36), 116), ((2, 9, 100, 16, 64), 100),
                                          ((2, 8, 31, 24, 68), 116), ((2, 5, 31, 24, 68), 100), ((3, 13, 11, 64, 64), 100), ((2, 3, 130, 32, 64), 100)])
def test_conv3x3_bwd_weight_fp32_patches_that_stick_out(shape, kernel):
    """fp32 weight gradient on patches that the image does not divide into (both widths), and sizes next to the line
    that keep linear tiles, against the oracle."""
    N, H, W, Cin, Cout = shape
    assert B.vgg_conv3x3_plan(B.PLAN_BWD_WEIGHT, B.F32, N, H, W, Cin, Cout)[0] == kernel
    _check_bwd_weight(B.F32, shape, seed=sum(shape) + 4)


@pytest.mark.parametrize("shape", [(37, 55, 16, 3, 8), (57, 9, 42, 3, 64), (9, 16, 48, 2, 16), (2, 224, 224, 3, 64)])
def test_conv3x3_bwd_weight_thin_layers_stay_inside_their_workspace(shape):
    # At most three input channels: fp32 takes a kernel with its own pixel tiling, hence its own number of
    # partial sums.  The workspace is exactly what the query asks for, followed by a guard that must survive.
    N, H, W, Cin, Cout = shape
    d = synth.conv_layer_inputs(N, H, W, Cin, Cout, seed=sum(shape) + 3)
    dw_ref, db_ref = R.conv3x3_bwd_weight(d["x"], d["dy"])
    for dtype in (B.F32, B.BF16):
        need = B.vgg_conv3x3_bwd_weight_workspace_bytes(dtype, N, H, W, Cin, Cout)
        buf = torch.full((need + 4096,), 0xA5, dtype=torch.uint8, device="cuda")
        cp = B.vgg_padded_channels(dtype, Cin)
        dwp = torch.full((9, Cout, cp), float("nan"), device="cuda")
        db = torch.empty((Cout,), device="cuda")
        B.vgg_conv3x3_bwd_weight(dtype, N, H, W, Cin, Cout, to_nhwc(d["x"], dtype), to_nhwc(d["dy"], dtype), dwp, db, buf[:need])
        torch.cuda.synchronize()
        assert (buf[need:] == 0xA5).all(), dtype
        dw = dwp[:, :, :Cin].reshape(3, 3, Cout, Cin).permute(2, 3, 0, 1)
        assert max_rel_err(dw.cpu().numpy(), dw_ref) <= TOL[dtype]
        assert max_rel_err(db.cpu().numpy(), db_ref) <= TOL[dtype]
        with pytest.raises(B.VggError):
            B.vgg_conv3x3_bwd_weight(dtype, N, H, W, Cin, Cout, to_nhwc(d["x"], dtype), to_nhwc(d["dy"], dtype), dwp, db,
                                     buf[:need - 256])


def test_paper_dense_and_softmax_examples():
    # The paper's two introductory functions at the sizes its compiled listings show: dense on a 10 x 10
    # matrix, a 10-vector and a 10-vector bias; softmax of a 10-vector (section "Two simple examples").
    rng = np.random.default_rng(1810)
    W = rng.standard_normal((10, 10)).astype(np.float32)
    x = rng.standard_normal((1, 10)).astype(np.float32)
    b = rng.standard_normal(10).astype(np.float32)
    z = torch.empty((1, 10), device="cuda")
    B.vgg_fc(B.F32, 1, 10, 10, dev(x), dev(W), dev(b), z, B.F32, 0, ws_bytes(B.vgg_fc_workspace_bytes(B.F32, 1, 10, 10)))
    p = torch.empty((1, 10), device="cuda")
    B.vgg_softmax(1, 10, z, p)
    torch.cuda.synchronize()
    zr = R.fc(x, W, b, relu=False)
    assert max_rel_err(z.cpu().numpy(), zr) <= 1e-6
    assert np.abs(z.cpu().numpy().astype(np.float64) - (W.astype(np.float64) @ x[0].astype(np.float64) + b)).max() <= 1e-5
    assert max_rel_err(p.cpu().numpy(), R.softmax(zr)) <= 1e-6
    assert abs(float(p.sum()) - 1.0) <= 1e-6


@pytest.mark.parametrize("shape", RANDOM_CONV_SHAPES)
def test_conv3x3_random_shapes(shape):
    for dtype in (B.F32, B.BF16):
        test_conv3x3_fwd(dtype, shape)
        test_conv3x3_bwd_data(dtype, shape)
    if shape[4] % 4 == 0:
        _check_bwd_weight(B.F32, shape, seed=sum(shape) + 2)
        _check_bwd_weight(B.BF16, shape, seed=sum(shape) + 2)


def test_pack_unpack_roundtrip_and_flip_layout():
    rng = np.random.default_rng(3)
    Cin, Cout = 5, 12
    w = rng.standard_normal((Cout, Cin, 3, 3)).astype(np.float32)
    p = _pack(B.F32, w)
    back = torch.empty((Cout, Cin, 3, 3), device="cuda")
    B.vgg_conv_unpack_weights(Cin, Cout, p, back)
    assert np.array_equal(back.cpu().numpy(), w)
    pf = _pack(B.F32, w, flip=1).cpu().numpy()       # [9][Cin][CoutP]
    for t in range(9):
        assert np.array_equal(pf[t, :, :Cout], w.reshape(Cout, Cin, 9)[:, :, 8 - t].T)
    assert not pf[:, :, Cout:].any()


@pytest.mark.parametrize("dtype", [B.F32, B.BF16])
@pytest.mark.parametrize("shape", [(2, 8, 12, 64), (3, 2, 2, 8), (1, 14, 14, 512)])
def test_maxpool_fwd_bwd(dtype, shape):
    N, H, W, Cc = shape
    rng = np.random.default_rng(sum(shape))
    x = rng.standard_normal((N, Cc, H, W)).astype(np.float32)
    xd = to_nhwc(x, dtype)
    xq = from_nhwc(xd)                        # what the kernel sees (bf16-rounded for BF16)
    p_ref, a_ref = R.maxpool2x2(xq)
    y = torch.empty((N, H // 2, W // 2, Cc), dtype=TDT[dtype], device="cuda")
    arg = torch.empty((N, H // 2, W // 2, Cc), dtype=torch.uint8, device="cuda")
    B.vgg_maxpool2x2(dtype, N, H, W, Cc, xd, y, arg)
    torch.cuda.synchronize()
    assert np.array_equal(from_nhwc(y), p_ref)                 # selection only: bit-exact
    a_gpu = arg.permute(0, 3, 1, 2).cpu().numpy()
    if dtype == B.F32:
        assert np.array_equal(a_gpu, a_ref)                    # random fp32 data has no ties
    else:
        # bf16 rounding creates ties; the oracle consumed the same rounded values, first-max rule applies
        assert np.array_equal(a_gpu, a_ref)
    dp = rng.standard_normal(p_ref.shape).astype(np.float32)
    dpd = to_nhwc(dp, dtype)
    dx = torch.full((N, H, W, Cc), float("nan"), dtype=TDT[dtype], device="cuda")
    B.vgg_maxpool2x2_bwd(dtype, N, H, W, Cc, dpd, arg, dx)
    torch.cuda.synchronize()
    assert np.array_equal(from_nhwc(dx), R.maxpool2x2_bwd(from_nhwc(dpd), a_ref))


def test_maxpool_ties_pick_first():
    x = np.zeros((1, 8, 4, 4), dtype=np.float32)
    x[0, 1] = 3.0
    x[0, 2, 1, 1] = 1.0
    xd = to_nhwc(x, B.F32)
    y = torch.empty((1, 2, 2, 8), device="cuda")
    arg = torch.empty((1, 2, 2, 8), dtype=torch.uint8, device="cuda")
    B.vgg_maxpool2x2(B.F32, 1, 4, 4, 8, xd, y, arg)
    _, a_ref = R.maxpool2x2(x)
    assert np.array_equal(arg.permute(0, 3, 1, 2).cpu().numpy(), a_ref)


@pytest.mark.parametrize("dtype", [B.F32, B.BF16])
@pytest.mark.parametrize("shape", [(100, 512, 1000), (2, 512, 10), (7, 2048, 96), (130, 64, 200),
                                   # rows that are not whole 64-byte units: the paper's own dense example
                                   # (a 10 x 10 matrix times a 10-vector, here also on ten vectors), odd
                                   # lengths, a last unit holding one element
                                   (1, 10, 10), (10, 10, 10), (3, 50, 7), (5, 37, 130), (129, 1, 3), (4, 8200, 40), (6, 2052, 9)])
def test_fc_forward(dtype, shape):
    N, In, Out = shape
    rng = np.random.default_rng(sum(shape))
    a = rng.standard_normal((N, In)).astype(np.float32)
    w = (rng.standard_normal((Out, In)) * np.sqrt(2.0 / In)).astype(np.float32)
    b = rng.standard_normal(Out).astype(np.float32)
    ws = ws_bytes(B.vgg_fc_workspace_bytes(dtype, N, In, Out))
    for relu, zdt in ((1, dtype), (0, B.F32)):
        ref = R.fc(a, w, b, relu=bool(relu))
        z = torch.empty((N, Out), dtype=TDT[zdt], device="cuda")
        B.vgg_fc(dtype, N, In, Out, dev(a, TDT[dtype]), dev(w, TDT[dtype]), dev(b), z, zdt, relu, ws)
        torch.cuda.synchronize()
        assert max_rel_err(z.float().cpu().numpy(), ref) <= TOL[dtype]


@pytest.mark.parametrize("dtype", [B.F32, B.BF16])
@pytest.mark.parametrize("shape", [(100, 512, 1000), (2, 512, 10), (7, 2048, 96), (130, 64, 200), (113, 160, 33), (250, 96, 72),
                                   (1, 10, 10), (10, 10, 10), (5, 37, 130), (9, 50, 64), (3, 1030, 5), (10, 24, 10)])
def test_fc_backward(dtype, shape):
    # bf16: a and w are bf16, dz fp32 (rounded to bf16 inside, except for db); all results fp32
    N, In, Out = shape
    if dtype == B.BF16 and In % 8:
        a = torch.zeros((64,), device="cuda")
        with pytest.raises(B.VggError):      # 16-byte segments of bf16 rows
            B.vgg_fc_bwd(dtype, N, In, Out, a, a, a, a, None, None, 0, a)
        return
    rng = np.random.default_rng(sum(shape) + 5)
    a = rng.standard_normal((N, In)).astype(np.float32)
    w = (rng.standard_normal((Out, In)) * np.sqrt(2.0 / In)).astype(np.float32)
    dz = rng.standard_normal((N, Out)).astype(np.float32)
    dw_ref, db_ref, da_ref = R.fc_bwd(a, w, dz)
    dw = torch.full((Out, In), float("nan"), device="cuda")
    db = torch.empty((Out,), device="cuda")
    da = torch.full((N, In), float("nan"), device="cuda")
    ws = ws_bytes(B.vgg_fc_bwd_workspace_bytes(dtype, N, In, Out))
    ad, wd = dev(a, TDT[dtype]), dev(w, TDT[dtype])
    B.vgg_fc_bwd(dtype, N, In, Out, ad, wd, dev(dz), dw, db, da, 0, ws)
    torch.cuda.synchronize()
    assert max_rel_err(dw.cpu().numpy(), dw_ref) <= TOL[dtype]
    assert max_rel_err(db.cpu().numpy(), db_ref) <= TOL[B.F32]         # a plain fp32 sum in both
    assert max_rel_err(da.cpu().numpy(), da_ref) <= TOL[dtype]
    B.vgg_fc_bwd(dtype, N, In, Out, ad, wd, dev(dz), dw, None, da, 1, ws)
    torch.cuda.synchronize()
    assert max_rel_err(da.cpu().numpy(), da_ref * (ad.float().cpu().numpy() > 0)) <= TOL[dtype]
    with pytest.raises(B.VggError):
        B.vgg_fc_bwd(dtype, N, In, Out, ad, wd, dev(dz), dw, None, da, 1, None)


@pytest.mark.parametrize("dtype", [B.F32, B.BF16])
@pytest.mark.parametrize("N,In,Out", [(1, 8, 3), (16, 264, 33), (17, 136, 130), (32, 520, 2050), (9, 4104, 16), (31, 2056, 17)])
def test_fc_forward_small_batches(dtype, N, In, Out):
    """The small-batch kernel at the edges of its tiles: one and two 16-row blocks, rows shorter than a 256-byte piece,
    pieces for more and for fewer than its sixteen waves, a ragged last tile of outputs.  Operands rounded to the dtype
    first, so that the sums (fp32, at most 4104 products) are all that differs: 1e-5 of the largest output."""
    rng = np.random.default_rng(N * In + Out)
    a, w = (dev(rng.standard_normal(s).astype(np.float32), TDT[dtype]) for s in ((N, In), (Out, In)))
    b = rng.standard_normal(Out).astype(np.float32)
    ref = R.fc(a.float().cpu().numpy(), w.float().cpu().numpy(), b, relu=True)
    z = torch.full((N * Out + 64,), -7.0, device="cuda")
    B.vgg_fc(dtype, N, In, Out, a, w, dev(b), z, B.F32, 1, ws_bytes(B.vgg_fc_workspace_bytes(dtype, N, In, Out)))
    torch.cuda.synchronize()
    assert max_rel_err(z[:N * Out].view(N, Out).cpu().numpy(), ref) <= 1e-5
    assert (z[N * Out:] == -7.0).all()


@pytest.mark.parametrize("dtype", [B.F32, B.BF16])
@pytest.mark.parametrize("N,In,Out", [(3, 10240, 16), (3, 10256, 16), (4, 49152, 16), (8, 49168, 9), (16, 20480, 40), (16, 30728, 40),
                                      (5, 28672, 64), (5, 28688, 70), (3, 40000, 10), (2, 22536, 600), (2, 8200, 3000), (24, 28680, 2048)])
def test_fc_forward_where_the_kernel_changes(dtype, N, In, Out):
    """Long rows on both sides of the lines between one workgroup per sixteen outputs and the split over workgroups,
    against the oracle on the operands as stored; 1e-5: fp32 sums of at most 49168 / 16 products in a row."""
    rng = np.random.default_rng(np.random.PCG64(N + In + Out))
    a, w = (dev(rng.standard_normal(s).astype(np.float32), TDT[dtype]) for s in ((N, In), (Out, In)))
    b = rng.standard_normal(Out).astype(np.float32)
    ref = R.fc(a.float().cpu().numpy(), w.float().cpu().numpy(), b, relu=False)
    z = torch.full((N * Out + 64,), -7.0, device="cuda")
    B.vgg_fc(dtype, N, In, Out, a, w, dev(b), z, B.F32, 0, ws_bytes(B.vgg_fc_workspace_bytes(dtype, N, In, Out)))
    torch.cuda.synchronize()
    assert max_rel_err(z[:N * Out].view(N, Out).cpu().numpy(), ref) <= 1e-5
    assert (z[N * Out:] == -7.0).all()


@pytest.mark.parametrize("dtype", [B.F32, B.BF16])
@pytest.mark.parametrize("N,In,Out", [(33, 264, 129), (64, 520, 127), (65, 136, 130), (96, 1032, 200), (97, 4104, 40), (128, 24, 257), (257, 264, 128),
                                      (40, 261, 65), (70, 1000, 33), (142, 22, 18), (70, 3, 5), (130, 37, 33),
                                      (3, 5120, 40), (3, 5136, 40), (16, 8704, 1500), (16, 8712, 1504), (2, 25608, 2504), (20, 3328, 96),
                                      (32, 3336, 96), (17, 8712, 2504), (20, 1664, 8200), (1, 2048, 8208),
                                      (5, 16388, 2052), (40, 16392, 2050), (9, 32776, 2056), (33, 32784, 2056)])
def test_fc_forward_row_blocks_and_streamed_weights(dtype, N, In, Out):
    """Every number of 32-row blocks of the split kernel, rows that end inside a step (whole 16-byte segments or not), both
    sides of the lines to the kernel of small batches, and weights of 128 MB, which are read past the caches; against the
    oracle on the operands as stored; 1e-5: fp32 sums of at most 32784 products in order."""
    rng = np.random.default_rng(np.random.PCG64(N + In + Out))
    a, w = (dev(rng.standard_normal(s, dtype=np.float32), TDT[dtype]) for s in ((N, In), (Out, In)))
    b = rng.standard_normal(Out).astype(np.float32)
    ref = R.fc(a.float().cpu().numpy(), w.float().cpu().numpy(), b, relu=False)
    z = torch.full((N * Out + 64,), -7.0, device="cuda")
    B.vgg_fc(dtype, N, In, Out, a, w, dev(b), z, B.F32, 0, ws_bytes(B.vgg_fc_workspace_bytes(dtype, N, In, Out)))
    torch.cuda.synchronize()
    assert max_rel_err(z[:N * Out].view(N, Out).cpu().numpy(), ref) <= 1e-5
    assert (z[N * Out:] == -7.0).all()


@pytest.mark.parametrize("N,In,Out", [(16, 260, 129), (17, 256, 64), (49, 1028, 3), (80, 132, 191), (97, 516, 257), (129, 252, 65),
                                      (31, 129, 1), (112, 127, 66), (40, 260, 129), (41, 256, 96), (48, 508, 33), (64, 1028, 160), (128, 100, 258), (41, 30, 5)])
def test_fc_backward_fp32_tile_edges(N, In, Out):
    """The fp32 backward kernels at the edges of their tiles (16-row blocks, 128- and 256-column tiles, 64-output
    passes, odd rows, rows that are not 16-byte aligned, both sides of the line to the bf16 matrix unit): sums of at most 257 (129) products of N(0,1) values against
    the oracle; the rounding of such a sum is below 1e-6 of the largest, the tolerance 1e-5."""
    rng = np.random.default_rng(N + In + Out)
    a, dz = rng.standard_normal((N, In)).astype(np.float32), rng.standard_normal((N, Out)).astype(np.float32)
    w = rng.standard_normal((Out, In)).astype(np.float32)
    dw_ref, db_ref, da_ref = R.fc_bwd(a, w, dz)
    dw, da = torch.full((Out * In + 256,), -7.0, device="cuda"), torch.full((N * In + 256,), -7.0, device="cuda")
    db = torch.empty((Out,), device="cuda")
    ws = ws_bytes(B.vgg_fc_bwd_workspace_bytes(B.F32, N, In, Out))
    B.vgg_fc_bwd(B.F32, N, In, Out, dev(a), dev(w), dev(dz), dw, db, da, 1, ws)
    torch.cuda.synchronize()
    assert max_rel_err(dw[:Out * In].view(Out, In).cpu().numpy(), dw_ref) <= 1e-5
    assert max_rel_err(da[:N * In].view(N, In).cpu().numpy(), da_ref * (a > 0)) <= 1e-5
    assert max_rel_err(db.cpu().numpy(), db_ref) <= 1e-5
    assert (dw[Out * In:] == -7.0).all() and (da[N * In:] == -7.0).all()


@pytest.mark.parametrize("N,In,Out,parts", [
    (25, 258, 1024, False), (24, 258, 1024, False), (32, 255, 1025, False), (41, 4097, 33, True), (57, 5002, 2602, True), (100, 2052, 5000, True),
    (128, 1026, 2600, False), (128, 6400, 1030, False), (129, 1026, 200, False),
    (40, 512, 1000, False), (50, 512, 4096, True), (50, 512, 4097, False),        # 40 and 41 rows; 256 and 258 units
    (70, 4096, 2048, False), (70, 4098, 2048, True), (128, 4225, 2050, True),     # 512 and 528 blocks
    (64, 4224, 2048, True), (64, 4232, 2048, False), (64, 4240, 2048, False), (64, 8464, 2048, True), (64, 4226, 2048, True),   # rows by alignment
])
def test_fc_backward_fp32_staged_gradient(N, In, Out, parts):
    """fp32 backward with dz taken apart ahead of the products (parts), and launches just outside the lines to it: workgroups
    of dW with one and with several (input tile, 32 outputs) units and with more than the four LDS buffers hold,
    of two input tiles, and ranges of outputs that end inside 32; every element against float64.  Sums of at most 5000 products of
    N(0,1) values in fp32 are within 1e-6 of the largest, the tolerance is 1e-5.  Guards behind the results, the workspace NaN before."""
    assert dz_in_parts(N, In, Out) == parts
    g = torch.Generator(device="cuda").manual_seed(N * In + Out)
    a, w, dz = (torch.randn(s, generator=g, device="cuda") for s in ((N, In), (Out, In), (N, Out)))
    dw, da = torch.full((Out * In + 256,), -7.0, device="cuda"), torch.full((N * In + 256,), -7.0, device="cuda")
    db = torch.empty((Out,), device="cuda")
    ws = ws_bytes(B.vgg_fc_bwd_workspace_bytes(B.F32, N, In, Out))
    ws.fill_(255)
    B.vgg_fc_bwd(B.F32, N, In, Out, a, w, dz, dw, db, da, 1, ws)
    torch.cuda.synchronize()
    a, w, dz = a.double(), w.double(), dz.double()
    for got, want in ((dw[:Out * In].view(Out, In), dz.t().contiguous() @ a), (db, dz.sum(0)), (da[:N * In].view(N, In), dz @ w * (a > 0))):
        assert ((got - want).abs().max() / want.abs().max()).item() <= 1e-5
    assert (dw[Out * In:] == -7.0).all() and (da[N * In:] == -7.0).all()


@pytest.mark.parametrize("N,In,Out", [(24, 258, 1024), (25, 258, 1024), (32, 255, 1025), (40, 1028, 2600), (41, 257, 1100), (57, 1030, 160),
                                      (100, 520, 2100), (128, 1026, 1024), (129, 136, 257), (200, 516, 130)])
def test_fc_backward_fp32_weight_gradient_alone(N, In, Out):
    """dW and db do not depend on whether da is asked for: the same bits with and without it, at batch sizes on both sides of every
    line between the kernels, and against float64 (tolerance as above)."""
    g = torch.Generator(device="cuda").manual_seed(N * In + Out)
    a, w, dz = (torch.randn(s, generator=g, device="cuda") for s in ((N, In), (Out, In), (N, Out)))
    got = []
    for da in (torch.empty((N, In), device="cuda"), None):
        dw, db = torch.full((Out * In + 256,), -7.0, device="cuda"), torch.empty((Out,), device="cuda")
        ws = None if da is None else ws_bytes(B.vgg_fc_bwd_workspace_bytes(B.F32, N, In, Out))
        B.vgg_fc_bwd(B.F32, N, In, Out, a, w, dz, dw, db, da, 1, ws)
        torch.cuda.synchronize()
        assert (dw[Out * In:] == -7.0).all()
        got.append((dw, db))
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])
    dw, want = got[1][0][:Out * In].view(Out, In), dz.double().t().contiguous() @ a.double()
    assert ((dw - want).abs().max() / want.abs().max()).item() <= 1e-5


@pytest.mark.parametrize("scale", [-116, 0, 100])
@pytest.mark.parametrize("N,In,Out", [(25, 260, 1024), (32, 256, 1024), (40, 255, 1026)])
def test_fc_backward_fp32_whole_range_up_to_40_rows(N, In, Out, scale):
    """Up to 40 batch rows the products are fp32 ones over the whole range of normal values: 1e-6 of the result's norm, six
    times what sums of at most 1026 products round off (1.6e-7; three bf16 parts per value: 4e-6 at 2^-116)."""
    g = torch.Generator(device="cuda").manual_seed(N * In + Out)
    a, w, dz = (torch.randn(s, generator=g, device="cuda") for s in ((N, In), (Out, In), (N, Out)))
    a, w = a * 2.0 ** scale, w * 2.0 ** scale
    dw, da = torch.empty((Out, In), device="cuda"), torch.empty((N, In), device="cuda")
    B.vgg_fc_bwd(B.F32, N, In, Out, a, w, dz, dw, None, da, 0, ws_bytes(B.vgg_fc_bwd_workspace_bytes(B.F32, N, In, Out)))
    torch.cuda.synchronize()
    for got, want in ((dw, dz.double().t().contiguous() @ a.double()), (da, dz.double() @ w.double())):
        err = ((got - want).norm() / want.norm()).item()
        print("relative error %.1e" % err)
        assert err <= 1e-6


@pytest.mark.parametrize("N,In,Out", [(41, 4097, 33), (64, 1026, 200), (96, 260, 1028), (100, 8192, 2048), (128, 130, 514)])
def test_fc_backward_fp32_workspace_of_partial_sums_only(N, In, Out):
    """A workspace that holds da's partial sums but not dz in parts (one sized for 200 rows at 8192 -> 2048, say) takes the kernels that
    split dz themselves: the same bits, nothing written past it; one of 256 bytes less is refused, before anything is written."""
    g = torch.Generator(device="cuda").manual_seed(N * In + Out)
    a, w, dz = (torch.randn(s, generator=g, device="cuda") for s in ((N, In), (Out, In), (N, Out)))
    full = B.vgg_fc_bwd_workspace_bytes(B.F32, N, In, Out)
    least = da_partial_sum_bytes(N, In, Out)
    assert dz_in_parts(N, In, Out)
    if (N, In, Out) == (100, 8192, 2048):
        assert least == B.vgg_fc_bwd_workspace_bytes(B.F32, 200, In, Out)
    got = []
    for size in (full, full - 256, least, least - 256):
        dw, db, da = (torch.full(s, -7.0, device="cuda") for s in ((Out, In), (Out,), (N, In)))
        ws = torch.full((full + 4096,), 255, dtype=torch.uint8, device="cuda")
        call = lambda: B.vgg_fc_bwd(B.F32, N, In, Out, a, w, dz, dw, db, da, 1, ws[:size])
        if size < least:
            with pytest.raises(B.VggError, match="workspace"):
                call()
        else:
            call()
        torch.cuda.synchronize()
        assert (ws[size:] == 255).all()
        got.append((dw, db, da))
    for other in got[1:3]:
        assert all(torch.equal(x, y) for x, y in zip(got[0], other))
    assert all((t == -7.0).all() for t in got[3])


@pytest.mark.parametrize("N,In,Out", [(1, 8, 1), (32, 136, 65), (33, 264, 129), (64, 128, 64), (65, 120, 63), (96, 1032, 200), (97, 40, 33),
                                      (128, 256, 130), (129, 136, 257)])
def test_fc_backward_bf16_row_blocks(N, In, Out):
    """The bf16 backward kernels with every number of 32-row blocks, at the edges of their tiles (64-output steps, 128-input
    tiles, 64-row passes).  All operands representable in bf16: fp32 sums of at most 257 products, 1e-5 of the largest."""
    rng = np.random.default_rng(N * 7 + In + Out)
    a, w, dz = (dev(rng.standard_normal(s).astype(np.float32), torch.bfloat16) for s in ((N, In), (Out, In), (N, Out)))
    dw_ref, db_ref, da_ref = R.fc_bwd(*(v.float().cpu().numpy() for v in (a, w, dz)))
    dw, da = torch.full((Out * In + 256,), -7.0, device="cuda"), torch.full((N * In + 256,), -7.0, device="cuda")
    db = torch.empty((Out,), device="cuda")
    B.vgg_fc_bwd(B.BF16, N, In, Out, a, w, dz.float(), dw, db, da, 1, ws_bytes(B.vgg_fc_bwd_workspace_bytes(B.BF16, N, In, Out)))
    torch.cuda.synchronize()
    assert max_rel_err(dw[:Out * In].view(Out, In).cpu().numpy(), dw_ref) <= 1e-5
    assert max_rel_err(da[:N * In].view(N, In).cpu().numpy(), da_ref * (a.float().cpu().numpy() > 0)) <= 1e-5
    assert max_rel_err(db.cpu().numpy(), db_ref) <= 1e-5
    assert (dw[Out * In:] == -7.0).all() and (da[N * In:] == -7.0).all()


def test_calls_go_to_the_current_stream():
    """The stream handed to the library is torch's current one: the default stream, a side stream, and again the default."""
    side = torch.cuda.Stream()
    assert B._stream() == torch.cuda.current_stream().cuda_stream
    with torch.cuda.stream(side):
        assert B._stream() == side.cuda_stream == torch.cuda.current_stream().cuda_stream
    assert B._stream() == torch.cuda.current_stream().cuda_stream != side.cuda_stream


@pytest.mark.parametrize("shape", [(100, 1000), (2, 10), (5, 64), (3, 129), (1, 10), (1, 1), (4, 5000)])
def test_softmax_xent_sgd(shape):
    N, K = shape
    rng = np.random.default_rng(N * K)
    z = (rng.standard_normal((N, K)) * 3).astype(np.float32)
    labels = rng.integers(0, K, size=N).astype(np.int32)
    p_ref = R.softmax(z)
    p = torch.empty((N, K), device="cuda")
    B.vgg_softmax(N, K, dev(z), p)
    torch.cuda.synchronize()
    assert max_rel_err(p.cpu().numpy(), p_ref) <= 1e-5
    loss_ref, dz_ref = R.softmax_xent(p.cpu().numpy().astype(np.float64), labels)
    loss = torch.empty((1,), device="cuda")
    dz = torch.empty((N, K), device="cuda")
    B.vgg_softmax_xent_bwd(N, K, p, dev(labels), loss, dz, ws_bytes(N * 4))
    torch.cuda.synchronize()
    assert abs(loss.item() - loss_ref) <= 1e-5 * abs(loss_ref)
    assert max_rel_err(dz.cpu().numpy(), dz_ref) <= 1e-6
    n = N * K + 3 if (N * K) % 4 else N * K - 1      # exercise the scalar tail
    theta = rng.standard_normal(n).astype(np.float32)
    grad = rng.standard_normal(n).astype(np.float32)
    th = dev(theta)
    B.vgg_sgd_update(n, th, dev(grad), 0.01)
    torch.cuda.synchronize()
    ref = R.sgd(theta, grad, 0.01)
    assert np.abs(th.cpu().numpy() - ref).max() <= 1e-6


@pytest.mark.parametrize("shape", [(301, 256), (7, 257), (303, 300), (5, 512), (5, 513), (3, 1024), (3, 1025), (2, 4096), (2, 4097)])
def test_softmax_xent_at_the_row_lengths_where_the_kernel_changes(shape):
    test_softmax_xent_sgd(shape)


def test_softmax_xent_with_more_rows_than_a_launch_has_workgroups():
    """2^24 rows: one more than a launch of a workgroup per row can have.  Softmax of 513 classes and the loss and
    gradient of 257, on rows that repeat a few patterns; the gradient alone of as many rows as a wavefront per row allows."""
    N = 1 << 24
    if torch.cuda.mem_get_info()[0] < 90 << 30:
        pytest.skip("needs 90 GB of device memory")
    rng = np.random.default_rng(24)
    for K in (513, 257):
        pat = (rng.standard_normal((64, K)) * 2).astype(np.float32)
        z = dev(pat).repeat(N // 64, 1)
        p = torch.empty_like(z)
        B.vgg_softmax(N, K, z, p)
        torch.cuda.synchronize()
        ref = R.softmax(pat)
        for r in (0, N // 2, N - 64):
            assert max_rel_err(p[r:r + 64].cpu().numpy(), ref) <= 1e-5
        if K == 257:
            labels = torch.from_numpy(rng.integers(0, K, size=64).astype(np.int32)).cuda().repeat(N // 64)
            loss = torch.zeros((1,), device="cuda")
            B.vgg_softmax_xent_bwd(N, K, p, labels, loss, z, ws_bytes(N * 4))
            torch.cuda.synchronize()
            loss_ref, dz_ref = R.softmax_xent(ref, labels[:64].cpu().numpy())
            # one lane adds 2^16 terms of about equal size one after another: at most 2^16 x 2^-24 of the sum
            assert abs(loss.item() - loss_ref) <= 4e-3 * abs(loss_ref)
            for r in (0, N // 2, N - 64):
                assert max_rel_err(z[r:r + 64].cpu().numpy() * (N / 64), dz_ref) <= 1e-6
        del z, p
        torch.cuda.empty_cache()
    N, K = (1 << 26) - 4, 2
    p = torch.full((N, K), 0.5, device="cuda")
    labels = torch.ones((N,), dtype=torch.int32, device="cuda")
    dz = torch.empty_like(p)
    loss = torch.zeros((1,), device="cuda")
    B.vgg_softmax_xent_bwd(N, K, p, labels, loss, dz, ws_bytes(N * 4))
    torch.cuda.synchronize()
    for r in (0, N // 3, N - 1):
        assert torch.equal((dz[r] * N).round(decimals=5).cpu(), torch.tensor([0.5, -0.5]))
    assert 0.6 < loss.item() < 0.8      # log 2, to the precision of that many equal terms in fp32
    torch.cuda.empty_cache()


def test_layout_roundtrip_and_convert():
    rng = np.random.default_rng(9)
    x = rng.standard_normal((2, 3, 6, 10)).astype(np.float32)
    y = torch.empty((2, 6, 10, 16), device="cuda")
    B.vgg_nchw_to_nhwc(B.F32, 2, 3, 6, 10, 16, dev(x), y)
    assert np.array_equal(y[..., :3].permute(0, 3, 1, 2).cpu().numpy(), x) and not y[..., 3:].any()
    back = torch.empty((2, 3, 6, 10), device="cuda")
    B.vgg_nhwc_to_nchw(B.F32, 2, 3, 6, 10, 16, y, back)
    assert np.array_equal(back.cpu().numpy(), x)
    # fp32 -> bf16 is round-to-nearest-even: torch implements the same IEEE rule
    v = dev(rng.standard_normal(1000).astype(np.float32))
    out = torch.empty((1000,), dtype=torch.bfloat16, device="cuda")
    B.vgg_convert(B.F32, B.BF16, 1000, v, out)
    assert torch.equal(out, v.to(torch.bfloat16))
    halfway = torch.tensor([1.00390625, 1.01171875], device="cuda")   # exactly between two bf16 values
    o2 = torch.empty((2,), dtype=torch.bfloat16, device="cuda")
    B.vgg_convert(B.F32, B.BF16, 2, halfway, o2)
    assert o2.float().tolist() == [1.0, 1.015625]                     # ties go to the even mantissa


def test_conv3x3_split_contraction_needs_its_workspace():
    # a shape whose contraction is split reports a workspace for the partial sums and refuses to run without it
    N, H, W, Cin, Cout = 1, 14, 14, 512, 512
    for dtype in (B.F32, B.BF16):
        need = B.vgg_conv3x3_fwd_workspace_bytes(dtype, N, H, W, Cin, Cout)
        assert need >= 2 * N * H * W * Cout * 4
        assert B.vgg_conv3x3_bwd_data_workspace_bytes(dtype, N, H, W, Cin, Cout) == need
        x = torch.zeros((N, H, W, Cin), dtype=TDT[dtype], device="cuda")
        w = torch.zeros((9, Cout, Cin), dtype=TDT[dtype], device="cuda")
        y = torch.empty((N, H, W, Cout), dtype=TDT[dtype], device="cuda")
        for ws in (None, ws_bytes(need - 256)):
            with pytest.raises(B.VggError):
                B.vgg_conv3x3_fwd(dtype, N, H, W, Cin, Cout, x, w, None, y, 1, ws)
            with pytest.raises(B.VggError):
                B.vgg_conv3x3_bwd_data(dtype, N, H, W, Cin, Cout, x, w, None, y, ws)
    # the batch-100 shapes keep every contraction in one workgroup: no workspace
    assert B.vgg_conv3x3_fwd_workspace_bytes(B.BF16, 100, 14, 14, 512, 512) == 0


def test_mfma_probe_runs_and_reports_flops():
    sink = torch.empty((B.vgg_mfma_probe_sink_bytes(),), dtype=torch.uint8, device="cuda")
    for dt, per in ((B.BF16, 2 * 32 * 32 * 16), (B.F32, 2 * 32 * 32 * 2)):
        flops = B.vgg_mfma_probe(dt, True, 10, sink)
        torch.cuda.synchronize()
        assert flops > 0 and flops % (10 * 8 * per) == 0
    # constant operands: every accumulator element is the contraction length times the MFMA count
    B.vgg_mfma_probe(B.BF16, False, 3, sink)
    torch.cuda.synchronize()
    vals = sink.view(torch.float32)[:256]
    assert torch.all(vals == 4 * 16 * (3 * 8 // 4) * 16.0)
    # the 16x16x32 shape: twice the instructions, each half the size, the same sums and the same operation count
    sink.zero_()
    assert B.vgg_mfma_probe(B.BF16, False, 3, sink, True) == B.vgg_mfma_probe(B.BF16, False, 3, sink)
    B.vgg_mfma_probe(B.BF16, False, 3, sink, True)
    torch.cuda.synchronize()
    assert torch.all(sink.view(torch.float32)[:256] == 4 * 16 * (3 * 8 // 4) * 16.0)
    with pytest.raises(B.VggError):
        B.vgg_mfma_probe(B.F32, False, 3, sink, True)
    small = torch.empty((16,), dtype=torch.uint8, device="cuda")
    with pytest.raises(B.VggError):
        B.vgg_mfma_probe(B.BF16, False, 3, small)
