"""GPU parity: every layer of the hot path, through the C ABI, against the CPU oracle.

Bit-exact for pack / unpack / max-pool / ReLU / add; |gpu - ref| <= 1e-4 (sqrt(K) max|ref| + 1)
for conv (K = Ci kh kw), depthwise and avg-pool (K = kh kw) and dense (K = Ci)."""
import numpy as np
import pytest
import torch

import paper_2303_04769_amd as S
from oracle import oracle as O
from gpu_util import CANARY, DEV, Guarded, assert_bits, assert_close, dev

pytestmark = pytest.mark.gpu


def _blk(C):
    return min(16, C)


# ------------------------------------------------------------------ layouts

@pytest.mark.parametrize("N,C,H,W,Cb", [(2, 32, 5, 7, 16), (1, 3, 96, 96, 3), (3, 8, 9, 13, 8), (2, 1, 49, 10, 1),
                                         (1, 64, 1, 1, 16), (2, 10, 1, 1, 10), (1, 48, 17, 9, 16), (1, 12, 3, 70, 4),
                                         (2, 32, 20, 20, 16), (1, 16, 16, 16, 16), (3, 64, 56, 56, 16), (2, 16, 8, 8, 16),
                                         (5, 48, 14, 14, 16), (1, 16, 2, 2, 16), (3, 16, 2, 2, 16), (7, 32, 3, 4, 16), (2, 16, 50, 50, 16)])
def test_pack_unpack_bit_exact(N, C, H, W, Cb):
    rng = np.random.default_rng(N * 1000 + C)
    x = rng.standard_normal((N, C, H, W)).astype(np.float32)
    g = Guarded(x.size)
    S.small_pack(dev(x), g.t, N, C, H, W, Cb)
    got = g.check()
    assert_bits(got, O.pack(x, Cb), "pack")
    g2 = Guarded(x.size)
    S.small_unpack(dev(got), g2.t, N, C, H, W, Cb)
    assert_bits(g2.check().reshape(x.shape), x, "unpack")


def test_pack_filters_bit_exact():
    rng = np.random.default_rng(3)
    for (Co, Ci, kh, kw, Cob, Cib) in [(32, 48, 3, 3, 16, 16), (16, 3, 3, 3, 16, 3), (64, 1, 10, 4, 16, 1),
                                       (10, 64, 1, 1, 10, 16), (16, 8, 1, 1, 16, 8)]:
        w = rng.standard_normal((Co, Ci, kh, kw)).astype(np.float32)
        g = Guarded(w.size)
        S.small_pack_filter(dev(w), g.t, Co, Ci, kh, kw, Cob, Cib)
        assert_bits(g.check(), O.pack_filter(w, Cob, Cib), "pack_filter")
    for (C, Cb) in [(32, 16), (8, 8), (3, 3)]:
        w = rng.standard_normal((C, 1, 3, 3)).astype(np.float32)
        g = Guarded(w.size)
        S.small_pack_dw_filter(dev(w), g.t, C, 3, 3, Cb)
        assert_bits(g.check(), O.pack_dw_filter(w, Cb), "pack_dw_filter")


# ------------------------------------------------------------------ single element

@pytest.mark.parametrize("n", [1, 3, 4, 1023, 4096, 16384, 100003])
def test_relu_add_bit_exact(n):
    rng = np.random.default_rng(n)
    a = rng.standard_normal(n).astype(np.float32)
    b = rng.standard_normal(n).astype(np.float32)
    special = np.array([-np.inf, -2.5, -0.0, 0.0, 1e-45, -1e-45, 3.0, np.inf, np.nan], np.float32)
    a[:min(n, special.size)] = special[:n]
    g = Guarded(n)
    S.small_relu(dev(a), g.t, n)
    assert_bits(g.check(), O.relu(a), "relu")
    g = Guarded(n)
    a2 = np.nan_to_num(a, nan=1.0, posinf=2.0, neginf=-2.0)
    S.small_add(dev(a2), dev(b), g.t, n)
    assert_bits(g.check(), O.add(a2, b), "add")
    # in place, and from an unaligned offset (scalar path)
    g = Guarded(n + 1)
    g.t[1:].copy_(dev(a))
    v = g.t[1:]
    S.small_relu(v, v, n)
    assert_bits(g.check()[1:], O.relu(a), "relu in place, unaligned")


# ------------------------------------------------------------------ convolution

def run_conv(x, w, stride, pad, Cib=None, Cob=None):
    N, Ci, H, W = x.shape
    Co, _, kh, kw = w.shape
    Cib, Cob = Cib or _blk(Ci), Cob or _blk(Co)
    xb, wb = dev(O.pack(x, Cib)), dev(O.pack_filter(w, Cob, Cib))
    Ho, Wo = O.out_dim(H, kh, stride, pad[0], pad[1]), O.out_dim(W, kw, stride, pad[2], pad[3])
    g = Guarded(N * Co * Ho * Wo)
    S.small_conv2d(xb, wb, g.t, N, Ci, Co, H, W, kh, kw, stride, pad, Cib, Cob)
    return O.unpack(g.check(), (N, Co, Ho, Wo), Cob)


CONV_CASES = [  # N, Ci, Co, H, W, kh, kw, stride, pad
    (1, 16, 16, 32, 32, 3, 3, 1, (1, 1, 1, 1)),      # the single-layer workload
    (3, 32, 48, 13, 11, 3, 3, 1, (1, 1, 1, 1)),      # ragged pixel tail, Co not a power of two
    (2, 64, 64, 9, 9, 1, 1, 1, (0, 0, 0, 0)),
    (2, 16, 32, 16, 16, 1, 1, 2, (0, 0, 0, 0)),      # projection shortcut
    (2, 16, 32, 32, 32, 3, 3, 2, (0, 1, 0, 1)),      # 'same' stride 2
    (3, 32, 32, 31, 31, 3, 3, 2, (1, 1, 1, 1)),      # stride 2, odd image, left / top padding
    (5, 48, 64, 20, 12, 3, 3, 2, (0, 1, 0, 1)),      # stride 2, non-square, three input-channel blocks
    (2, 16, 32, 32, 32, 3, 3, 2, (1, 1, 1, 1)),      # stride 2 whose last tap stays inside the image
    (4, 64, 32, 15, 15, 1, 1, 2, (0, 0, 0, 0)),      # 1x1 stride 2, odd image, two planes per step
    (2, 16, 16, 9, 9, 1, 1, 3, (0, 0, 0, 0)),        # 1x1 stride 3
    (1, 32, 16, 7, 9, 5, 3, 2, (2, 2, 1, 1)),        # odd window
    (2, 16, 16, 6, 6, 3, 3, 1, (0, 0, 0, 0)),        # no padding
    (4, 256, 128, 7, 7, 3, 3, 1, (1, 1, 1, 1)),      # pixel groups straddle images, a long reduction
    (2, 1, 64, 49, 10, 10, 4, 2, (4, 5, 1, 1)),      # generic path: Ci = 1
    (2, 3, 16, 32, 32, 3, 3, 1, (1, 1, 1, 1)),       # generic path: Ci = 3
    (1, 3, 8, 96, 96, 3, 3, 2, (0, 1, 0, 1)),        # generic path: 8-channel output block
    (2, 8, 16, 24, 24, 1, 1, 1, (0, 0, 0, 0)),       # generic path: 8-channel input block
    (5, 64, 10, 1, 1, 1, 1, 1, (0, 0, 0, 0)),        # generic path: dense-like head
    (3, 16, 10, 4, 5, 4, 5, 1, (0, 0, 0, 0)),        # dense over a 4 x 5 image (window = image)
]


@pytest.mark.parametrize("case", CONV_CASES)
def test_conv2d(case):
    N, Ci, Co, H, W, kh, kw, s, pad = case
    rng = np.random.default_rng(abs(hash(case)) % 2**31)
    x = (rng.random((N, Ci, H, W), dtype=np.float32) * 2 - 1).astype(np.float32)
    w = (rng.random((Co, Ci, kh, kw), dtype=np.float32) * 2 - 1).astype(np.float32)
    got = run_conv(x, w, s, pad)
    assert_close(got, O.conv2d(x, w, s, pad), Ci * kh * kw, f"conv {case}")


def test_conv2d_large_tiles():
    """Layers that fill the chip several times over, whatever kernel takes them (SAME_TILE_CASES go by kernel and tile)."""
    rng = np.random.default_rng(77)
    for Ci, Co, N, H in [(32, 128, 18, 45), (16, 64, 10, 58), (16, 32, 9, 61), (16, 16, 9, 61)]:
        x = (rng.random((N, Ci, H, H), dtype=np.float32) * 2 - 1).astype(np.float32)
        w = (rng.random((Co, Ci, 3, 3), dtype=np.float32) * 2 - 1).astype(np.float32)
        got = run_conv(x, w, 1, (1, 1, 1, 1))
        assert_close(got, O.conv2d(x, w, 1, (1, 1, 1, 1)), Ci * 9, f"conv large {Ci}->{Co}")


SAME_TILE_CASES = [  # N, Ci, Co, H, W, k, stride, pad, kernel: every tile that 3x3 and 1x1 layers have in conv_same.hip
    (4, 16, 112, 25, 6, 3, 1, (1, 1, 1, 1), "conv16_same<4,1,1,1,3,1,1>"),        # 64 x 16; odd rows; tiles across images
    (15, 16, 128, 23, 6, 3, 1, (1, 1, 1, 1), "conv16_same<4,1,1,2,3,1,1>"),       # 64 x 32
    (6, 80, 144, 25, 27, 3, 1, (1, 1, 1, 1), "conv16_same<4,1,1,1,3,1,1>"),       # five input blocks, nine output blocks
    (13, 16, 96, 19, 11, 3, 1, (1, 1, 1, 1), "conv16_same<2,2,1,1,3,1,1>"),       # 32 x 32; tiles across images, odd images
    (11, 16, 16, 39, 41, 3, 1, (1, 1, 1, 1), "conv16_same<4,1,2,1,3,1,1>"),       # 128 x 16, one output block
    (2, 16, 256, 13, 37, 3, 2, (1, 1, 1, 1), "conv16_same<4,1,1,1,3,1,2>"),       # stride 2, odd images
    (226, 16, 64, 13, 5, 3, 2, (1, 1, 1, 1), "conv16_same<4,1,1,2,3,1,2>"),       # ... 21 output pixels an image
    (54, 32, 16, 33, 55, 3, 2, (1, 1, 1, 1), "conv16_same<4,1,2,1,3,1,2>"),
    (3, 80, 96, 59, 59, 3, 2, (1, 1, 1, 1), "conv16_same<2,2,1,1,3,1,2>"),
    (46, 16, 240, 13, 14, 3, 1, (1, 1, 1, 1), "conv16_img<4,1,1,1,3,1,1>"),       # tiles end with the image: 182 pixels
    (7, 16, 240, 37, 55, 3, 1, (1, 1, 1, 1), "conv16_img<4,1,1,2,3,1,1>"),        # fifteen output blocks under tiles of two
    (5, 16, 32, 7, 3, 1, 3, (0, 0, 0, 0), "conv16_same<2,2,1,1,1,1,1>"),          # 1x1, one input block, stride 3
    (2, 32, 48, 5, 37, 1, 2, (0, 0, 0, 0), "conv16_same<2,2,1,1,1,2,1>"),         # two planes a step, three output blocks
    (5, 16, 80, 9, 3, 1, 2, (0, 0, 0, 0), "conv16_same<2,2,1,2,1,1,1>"),          # 32 x 64, five output blocks
    (2, 64, 64, 3, 22, 1, 2, (0, 0, 0, 0), "conv16_same<2,2,1,2,1,2,1>"),
    (2, 16, 16, 7, 16, 1, 1, (0, 0, 0, 0), "conv16_same<4,1,1,1,1,1,1>"),         # 64 x 16, 1x1
    (2, 32, 16, 9, 12, 1, 2, (0, 0, 0, 0), "conv16_same<4,1,1,1,1,2,1>"),
]


@pytest.mark.parametrize("case", SAME_TILE_CASES)
def test_conv2d_same_tiles(case):
    N, Ci, Co, H, W, k, s, pad, kernel = case
    assert S.small_conv2d_kernel(N, Ci, Co, H, W, k, k, s, pad, 16, 16) == kernel, case
    rng = np.random.default_rng(8700 + N + Co)
    x = (rng.random((N, Ci, H, W), dtype=np.float32) * 2 - 1).astype(np.float32)
    w = (rng.random((Co, Ci, k, k), dtype=np.float32) * 2 - 1).astype(np.float32)
    assert_close(run_conv(x, w, s, pad), O.conv2d(x, w, s, pad), Ci * k * k, f"conv tile {case}")


STRIDED_CASES = [  # N, Ci, Co, H, W, pad, kernel: 3x3 with stride 2, tiles of three output blocks, and images whose rows' last tap is inside
    (50, 16, 96, 45, 37, (1, 1, 1, 1), "conv16_same<4,1,1,3,3,1,2>"),          # 64 x 48; tap 0 of a row's first pixel outside, tap 2 of its last
    (176, 16, 224, 17, 11, (1, 1, 1, 1), "conv16_same<4,1,1,3,3,1,2>"),        # fourteen output blocks under tiles of three
    (124, 16, 80, 17, 11, (1, 1, 1, 1), "conv16_same<4,1,1,1,3,1,2>"),         # no more such tiles than compute units: smaller ones
    (78, 16, 48, 44, 32, (0, 1, 0, 1), "conv16_same<4,1,1,3,3,1,2>"),          # padded on the right only
    (50, 32, 96, 45, 36, (1, 1, 1, 1), "conv16_same<4,1,1,2,3,1,3>"),          # tap 2 of a row's last pixel inside; tiles across images
    (159, 32, 48, 45, 62, (1, 1, 1, 1), "conv16_same<4,1,1,3,3,1,3>"),         # ... 64 x 48
    (150, 32, 80, 32, 30, (1, 1, 1, 0), "conv16_img<4,1,1,1,3,1,3>"),          # ... 64 x 16, tiles end with the image
    (161, 32, 96, 16, 35, (0, 1, 1, 0), "conv16_same<4,1,1,3,3,1,3>"),         # ... padded on the left only, rows from the image's first
    (110, 32, 48, 33, 64, (2, 1, 2, 1), "conv16_same<4,1,1,3,3,1,2>"),         # padded by two: taps 0 and 1 outside, tap 2 of the last too
    (113, 32, 48, 33, 63, (2, 1, 2, 1), "conv16_same<4,1,1,3,3,1,3>"),         # ... padded by two: taps 0 and 1 outside
    (300, 32, 16, 44, 38, (1, 1, 1, 1), "conv16_same<4,1,2,1,3,1,3>"),         # ... one output block
    (130, 32, 48, 32, 32, (1, 1, 1, 1), "conv16_same<4,1,1,1,3,1,3>"),         # ... just over 24 tiles per compute unit
    (64, 48, 64, 32, 32, (1, 1, 1, 1), "conv16_split<4,2,2>"),                 # ... and below
    (71, 96, 96, 43, 44, (1, 1, 1, 1), "conv16_split<2,2,2,taps>"),            # ... tiles of one block that would end with the image
    (150, 16, 96, 45, 36, (1, 1, 1, 1), "conv16_mfma<4,1,1,2>"),               # ... one input block
]


@pytest.mark.parametrize("case", STRIDED_CASES)
def test_conv2d_strided(case):
    N, Ci, Co, H, W, pad, kernel = case
    assert S.small_conv2d_kernel(N, Ci, Co, H, W, 3, 3, 2, pad, 16, 16) == kernel, case
    rng = np.random.default_rng(8800 + N + W)
    x = (rng.random((N, Ci, H, W), dtype=np.float32) * 2 - 1).astype(np.float32)
    w = (rng.random((Co, Ci, 3, 3), dtype=np.float32) * 2 - 1).astype(np.float32)
    assert_close(run_conv(x, w, 2, pad), O.conv2d(x, w, 2, pad), Ci * 9, f"strided {case}")


PERSISTENT_CASES = [  # N, Ci, Co, H, W, k: enough images that a workgroup walks several of them
    (131, 16, 16, 32, 32, 3),      # 16 tiles per image, last image group ragged
    (160, 16, 16, 30, 30, 3),      # image size not a multiple of the tile: masked lanes in each image's last tile
    (240, 16, 32, 24, 24, 3),      # 24 x 24 images: 9 full tiles, two output-channel blocks per wave
    (48, 32, 48, 40, 40, 3),       # three channel tiles per pixel tile
    (150, 16, 32, 48, 48, 3, 2),   # stride 2: two staged entries per output pixel
    (256, 16, 16, 32, 32, 3),      # the 128-pixel tile of the residual network's first stage at batch 256
]


@pytest.mark.parametrize("case", PERSISTENT_CASES)
def test_conv2d_persistent_variant(case):
    """Image-aligned persistent kernel: same results as the definition, and it really is the one that runs."""
    N, Ci, Co, H, W, k = case[:6]
    stride = case[6] if len(case) > 6 else 1
    pad = ((1, 1, 1, 1) if stride == 1 else (0, 1, 0, 1)) if k == 3 else (0, 0, 0, 0)
    assert S.small_conv2d_kernel(N, Ci, Co, H, W, k, k, stride, pad, 16, 16).startswith("conv16_img"), case
    rng = np.random.default_rng(1000 + N)
    x = (rng.random((N, Ci, H, W), dtype=np.float32) * 2 - 1).astype(np.float32)
    w = (rng.random((Co, Ci, k, k), dtype=np.float32) * 2 - 1).astype(np.float32)
    got = run_conv(x, w, stride, pad)
    assert_close(got, O.conv2d(x, w, stride, pad), Ci * k * k, f"conv persistent {case}")


POINTWISE_STREAM_CASES = [  # N, C, H, W: 64 or 128 channels, at least 32768 pixels
    (3, 64, 105, 105),       # 33075 pixels: groups of 16 straddle images, the last group has 3 pixels
    (70, 64, 25, 19),        # 33250 pixels, many small images, ragged end (2 pixels)
    (11, 128, 55, 55),       # 128 channels: two waves share a pixel group; 33275 pixels (11 in the last group)
    (9, 128, 61, 60),        # 32940 pixels: a tail of units after the full rounds
    (16, 64, 64, 64),        # 65536 pixels: 4096 groups = 2 full rounds on 2048 waves, no tail, no ragged group
    (17, 64, 64, 64),        # ... and one image more: a short tail
    (40, 128, 30, 30),       # 36000 pixels = 2250 groups: fewer tasks than two rounds of 512 tasks
]


@pytest.mark.parametrize("case", POINTWISE_STREAM_CASES)
def test_conv2d_pointwise_stream(case):
    """1x1 convolutions on 64 / 128 channels with many pixels run in the persistent kernel with the filter resident
    (asserted by name): full rounds of tasks, the finer units of the tail, and the ragged last group."""
    N, C, H, W = case
    name = S.small_conv2d_kernel(N, C, C, H, W, 1, 1, 1, (0, 0, 0, 0), 16, 16)
    assert name.startswith("pw16_stream"), (case, name)
    rng = np.random.default_rng(6100 + N + C)
    x = (rng.random((N, C, H, W), dtype=np.float32) * 2 - 1).astype(np.float32)
    w = (rng.random((C, C, 1, 1), dtype=np.float32) * 2 - 1).astype(np.float32)
    got = run_conv(x, w, 1, (0, 0, 0, 0))
    assert_close(got, O.conv2d(x, w, 1, (0, 0, 0, 0)), C, f"pointwise stream {case}")


FIRST_LAYER_CASES = [  # N, Ci, Co, H, W, kh, kw, stride, pad: at least 16384 output pixels, one short input block
    (17, 3, 16, 32, 32, 3, 3, 1, (1, 1, 1, 1)),      # K = 27: the residual network's first layer, ragged pixel tail
    (8, 3, 8, 96, 96, 3, 3, 2, (0, 1, 0, 1)),        # 8-channel output block, stride 2, bottom / right padding
    (140, 1, 64, 49, 10, 10, 4, 2, (4, 5, 1, 1)),    # K = 40: the audio network's first layer, four output blocks
    (20, 1, 16, 30, 31, 5, 5, 1, (2, 2, 2, 2)),      # K = 25 (padded to 28), wide padding on all sides
    (5, 2, 32, 60, 61, 2, 7, 1, (0, 1, 3, 3)),       # K = 28 exactly, two input channels
    (9, 5, 16, 44, 45, 2, 4, 1, (1, 0, 2, 1)),       # K = 40 with five input channels
    (3, 3, 16, 80, 81, 13, 1, 1, (6, 6, 0, 0)),      # K = 39: a tall window
    (40, 8, 16, 24, 24, 1, 1, 1, (0, 0, 0, 0)),      # K = 8: the pointwise layer after the 8-channel depthwise one
    (12, 2, 8, 40, 41, 2, 2, 1, (0, 1, 1, 0)),       # K = 8 from a 2 x 2 window of two channels
    (30, 5, 16, 30, 30, 1, 1, 1, (0, 0, 0, 0)),      # K = 5 (padded to 8)
]


@pytest.mark.parametrize("case", FIRST_LAYER_CASES)
def test_conv2d_first_layer_matrix_core(case):
    N, Ci, Co, H, W, kh, kw, s, pad = case
    name = S.small_conv2d_kernel(N, Ci, Co, H, W, kh, kw, s, pad, Ci, _blk(Co))
    assert name.startswith("conv_first_mfma"), (case, name)
    rng = np.random.default_rng(4000 + N)
    x = (rng.random((N, Ci, H, W), dtype=np.float32) * 2 - 1).astype(np.float32)
    w = (rng.random((Co, Ci, kh, kw), dtype=np.float32) * 2 - 1).astype(np.float32)
    got = run_conv(x, w, s, pad)
    assert_close(got, O.conv2d(x, w, s, pad), Ci * kh * kw, f"first layer {case}, all {N} images")


FIRST_LAYER_FEW_CASES = [  # N, Ci, Co, H, W, kh, kw, stride, pad: fewer than 16384 output pixels
    (1, 3, 16, 32, 32, 3, 3, 1, (1, 1, 1, 1)),       # 1024 pixels: 16 workgroups of 64
    (1, 3, 8, 96, 96, 3, 3, 2, (0, 1, 0, 1)),        # 8-channel output block
    (3, 1, 64, 49, 10, 10, 4, 2, (4, 5, 1, 1)),      # four output blocks; 375 pixels: a ragged last group
    (1, 3, 32, 1, 1, 3, 3, 1, (1, 1, 1, 1)),         # one pixel
    (2, 8, 16, 7, 9, 1, 1, 1, (0, 0, 0, 0)),         # K = 8
    (2, 5, 16, 11, 6, 2, 4, 1, (1, 0, 2, 1)),        # K = 40, five channels
    (130, 3, 16, 11, 11, 3, 3, 1, (1, 1, 1, 1)),     # 15730 pixels: just below the limit
    (1, 3, 512, 9, 9, 3, 3, 1, (1, 1, 1, 1)),        # every output block a workgroup of its own
    (24, 8, 1008, 24, 24, 1, 1, 1, (0, 0, 0, 0)),    # 63 output blocks in two shares, the second one short
    (64, 1, 112, 49, 10, 10, 4, 2, (4, 5, 1, 1)),    # seven in four shares, the last one block
]


@pytest.mark.parametrize("case", FIRST_LAYER_FEW_CASES)
def test_conv2d_first_layer_few_pixels(case):
    N, Ci, Co, H, W, kh, kw, s, pad = case
    name = S.small_conv2d_kernel(N, Ci, Co, H, W, kh, kw, s, pad, Ci, _blk(Co))
    assert name.startswith("conv_first_mfma") and name.endswith(",1>"), (case, name)
    rng = np.random.default_rng(4300 + N)
    x = (rng.random((N, Ci, H, W), dtype=np.float32) * 2 - 1).astype(np.float32)
    w = (rng.random((Co, Ci, kh, kw), dtype=np.float32) * 2 - 1).astype(np.float32)
    got = run_conv(x, w, s, pad)
    assert_close(got, O.conv2d(x, w, s, pad), Ci * kh * kw, f"first layer {case}")


@pytest.mark.parametrize("case", FIRST_LAYER_FEW_CASES)
def test_conv2d_first_layer_few_pixels_infinite_weights(case):
    """A tap outside the image does not count, whatever its weight: infinite and NaN weights at corners of the window, in one
    channel each; an infinite input value reaches the outputs whose window holds it."""
    N, Ci, Co, H, W, kh, kw, s, pad = case
    rng = np.random.default_rng(4350 + N)
    x = (rng.random((N, Ci, H, W), dtype=np.float32) + 1).astype(np.float32)
    w = (rng.random((Co, Ci, kh, kw), dtype=np.float32) + 1).astype(np.float32)
    w[1, 0, 0, 0], w[2, Ci - 1, kh - 1, kw - 1], w[Co - 1, 0, 0, kw - 1] = np.inf, np.nan, -np.inf
    x[0, 0, 0, 0] = np.inf
    got, ref = run_conv(x, w, s, pad), O.conv2d(x, w, s, pad)
    ok = np.isfinite(ref)
    assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.array_equal(got[~ok], ref[~ok], equal_nan=True)
    if (pad[0] or pad[2]) and H > 1:
        assert ok[:, 1].any() and not ok[:, 1].all()
    # sums of K positive products, every partial sum below the result: at most K roundings of 2^-24 of it
    assert (np.abs(got[ok].astype(np.float64) - ref[ok]) <= Ci * kh * kw * 2.0 ** -23 * np.abs(ref[ok])).all()


SPLIT_CASES = [  # N, Ci, Co, H, W, kh, kw, stride, pad, kernel: the reduction split over the waves of a workgroup
    (1, 512, 48, 6, 6, 3, 3, 1, (1, 1, 1, 1), "16,1,1"),       # 288 steps, 36 pixels: a ragged third pixel group
    (2, 80, 80, 6, 94, 5, 5, 2, (2, 2, 2, 2), "8,1,1"),        # 125 steps
    (1, 96, 16, 1, 1, 3, 3, 1, (1, 1, 1, 1), "4,1,1"),         # one pixel, eight of nine taps outside
    (5, 16, 32, 9, 7, 2, 2, 1, (1, 0, 0, 1), "4,1,1"),         # 4 steps: one per wave; a window without a middle
    (3, 32, 48, 23, 11, 3, 3, 3, (2, 1, 0, 2), "4,1,1"),       # stride 3, uneven padding
    (20, 16, 16, 68, 68, 3, 3, 2, (1, 1, 1, 1), "4,2,1"),      # one output block, many pixels
    (12, 32, 48, 70, 70, 3, 3, 2, (1, 1, 1, 1), "4,2,2"),      # three output blocks: the last workgroup has one
    (31, 16, 112, 59, 60, 4, 4, 2, (1, 1, 1, 1), "2,2,2"),     # seven output blocks; pixels end inside a group
    (7, 64, 48, 41, 41, 2, 2, 1, (1, 1, 1, 1), "4,2,2"),       # runs of four steps, four in flight; three output blocks
    (94, 128, 80, 14, 14, 2, 2, 1, (1, 1, 1, 1), "2,2,2"),     # ... of sixteen
    # taps innermost: a large input, strided, or many output blocks on it
    (23, 368, 16, 33, 25, 3, 3, 2, (1, 1, 1, 1), "16,1,1,taps"),    # 207 steps, 13 a wave: runs start inside a block
    (25, 208, 16, 31, 27, 3, 3, 2, (1, 1, 1, 1), "8,1,1,taps"),     # 117 steps, 15 a wave; the last has 12
    (31, 208, 112, 29, 23, 3, 2, 3, (0, 2, 1, 1), "4,1,1,taps"),    # stride 3, uneven padding; a window without a middle
    (45, 96, 80, 32, 27, 2, 3, 2, (1, 0, 0, 2), "4,2,2,taps"),      # five output blocks, 36 steps
    (212, 64, 64, 42, 7, 2, 2, 2, (1, 1, 1, 1), "4,2,2,taps"),      # runs of four steps, four in flight
    (140, 112, 96, 27, 17, 1, 3, 2, (0, 0, 1, 1), "2,2,2,taps"),    # 21 steps on two waves: eleven and ten
    (50, 256, 272, 14, 13, 1, 2, 1, (0, 0, 0, 0), "2,2,2,taps"),    # stride 1, seventeen output blocks
    (150, 160, 16, 40, 41, 3, 3, 3, (0, 0, 0, 0), "4,2,1,taps"),    # one output block
]


@pytest.mark.parametrize("case", SPLIT_CASES)
def test_conv2d_split_reduction(case):
    N, Ci, Co, H, W, kh, kw, s, pad, variant = case
    assert S.small_conv2d_kernel(N, Ci, Co, H, W, kh, kw, s, pad, 16, 16) == f"conv16_split<{variant}>", case
    rng = np.random.default_rng(8100 + N + Ci)
    x = (rng.random((N, Ci, H, W), dtype=np.float32) * 2 - 1).astype(np.float32)
    w = (rng.random((Co, Ci, kh, kw), dtype=np.float32) * 2 - 1).astype(np.float32)
    got = run_conv(x, w, s, pad)
    assert_close(got, O.conv2d(x, w, s, pad), Ci * kh * kw, f"conv split {case}")


def test_conv2d_split_reduction_infinities():
    """An infinite filter value in the first step and an infinite input value reach the outputs that contain them and no
    other: what a wave multiplies past its last step is zero by zero."""
    rng = np.random.default_rng(8200)
    x = (rng.random((1, 32, 5, 5), dtype=np.float32) + 1).astype(np.float32)
    w = (rng.random((32, 32, 3, 3), dtype=np.float32) + 1).astype(np.float32)
    w[3, 0, 0, 0] = np.inf
    x[0, 17, 4, 4] = -np.inf
    assert S.small_conv2d_kernel(1, 32, 32, 5, 5, 3, 3, 1, (0, 0, 0, 0), 16, 16).startswith("conv16_split")
    got = run_conv(x, w, 1, (0, 0, 0, 0))
    assert (got[0, 3].reshape(-1)[:8] == np.inf).all() and np.isnan(got[0, 3, 2, 2])
    rest = np.delete(got[0], 3, axis=0)
    assert (rest[:, 2, 2] == -np.inf).all() and np.isfinite(rest.reshape(31, 9)[:, :8]).all()


SPLIT3_CASES = [  # N, Ci, Co, H, W, kh, kw, pad: stride 1, at least 240 tiles of 128 pixels x 64 channels
    (40, 32, 64, 28, 28, 3, 3, (1, 1, 1, 1)),        # one chunk of two input blocks
    (34, 32, 112, 29, 31, 3, 3, (1, 1, 1, 1)),       # seven output blocks; two strips, the second a column short; ragged end
    (640, 64, 64, 7, 7, 3, 3, (1, 1, 1, 1)),         # tiles over three images
    (24, 16, 64, 37, 35, 5, 5, (2, 2, 2, 2)),        # one input block: two taps a step, the last step has one
    (23, 48, 64, 53, 50, 2, 4, (1, 0, 0, 3)),        # an odd input block, a window without a middle, uneven padding
    (40, 112, 64, 30, 30, 3, 3, (0, 0, 0, 0)),       # seven input blocks, no padding
]


@pytest.mark.parametrize("case", SPLIT3_CASES)
@pytest.mark.parametrize("scale", [1.0, 1e-36, 1e18, 1e30])
def test_conv2d_three_part_products(case, scale):
    """scale: where the parts of a value would be denormal, and where the sums overflow at the scale of the parts."""
    N, Ci, Co, H, W, kh, kw, pad = case
    assert S.small_conv2d_kernel(N, Ci, Co, H, W, kh, kw, 1, pad, 16, 16).startswith("conv16_split3"), case
    rng = np.random.default_rng(8300 + N + Ci)
    x = ((rng.random((N, Ci, H, W), dtype=np.float32) * 2 - 1) * np.float32(scale)).astype(np.float32)
    w = (rng.random((Co, Ci, kh, kw), dtype=np.float32) * 2 - 1).astype(np.float32)
    got = run_conv(x, w, 1, pad)
    idx = np.r_[0, 1, N // 2, N - 1]
    ref = O.conv2d(x[idx], w, 1, pad)
    # K products of 24-bit operands, what the three parts drop (up to 2^-24 of each) and the fp32 sums: below K 2^-24 of the largest
    bound = Ci * kh * kw * 2.0 ** -24 * scale
    assert np.isfinite(got).all() and np.abs(got[idx].astype(np.float64) - ref).max() <= bound + 2.0 ** -22 * np.abs(ref).max()


GATHER_CASES = [  # N, Ci, Co, H, W, kh, kw, stride, pad, kernel: short reductions under windows that have no tiles of their own
    (1, 16, 16, 5, 5, 1, 2, 1, (0, 0, 0, 0), "4,1,1,1"),       # 2 steps, 20 pixels of a tile of 64
    (7, 16, 32, 19, 23, 1, 3, 1, (0, 0, 1, 1), "4,1,1,1"),     # tiles across images
    (3, 16, 144, 39, 37, 3, 1, 2, (1, 1, 0, 0), "4,1,1,1"),    # nine output blocks
    (40, 16, 16, 25, 27, 2, 2, 1, (1, 0, 0, 1), "4,1,2,1"),    # uneven padding, one output block
    (9, 48, 96, 40, 41, 1, 2, 2, (0, 0, 0, 1), "4,1,1,2"),     # 6 steps on 27 tiles a compute unit
    (15, 80, 240, 66, 65, 1, 3, 2, (0, 0, 0, 2), "4,1,1,2"),   # 15 steps; fifteen output blocks: the last tile has one
    (31, 16, 112, 59, 60, 3, 3, 2, (1, 1, 1, 1), "4,1,1,1"),   # 9 steps: 19.0 us, with the reduction split 26.2
    (20, 16, 96, 9, 16, 1, 2, 1, (0, 0, 0, 0), "2,2,1,1"),
    (45, 32, 64, 86, 92, 3, 3, 3, (1, 1, 1, 1), "4,1,1,2"),    # 18 steps, 24 with the last round filled up
]


@pytest.mark.parametrize("case", GATHER_CASES)
def test_conv2d_gather_kernel(case):
    N, Ci, Co, H, W, kh, kw, s, pad, tile = case
    assert S.small_conv2d_kernel(N, Ci, Co, H, W, kh, kw, s, pad, 16, 16) == f"conv16_mfma<{tile}>", case
    rng = np.random.default_rng(8600 + N + Ci)
    x = (rng.random((N, Ci, H, W), dtype=np.float32) * 2 - 1).astype(np.float32)
    w = (rng.random((Co, Ci, kh, kw), dtype=np.float32) * 2 - 1).astype(np.float32)
    got = run_conv(x, w, s, pad)
    idx = np.unique(np.r_[0, N // 2, N - 1])
    assert np.isfinite(got).all()
    assert_close(got[idx], O.conv2d(x[idx], w, s, pad), Ci * kh * kw, f"conv gather {case}")


@pytest.mark.parametrize("N,Ci,Co,H,W,k,tile", [
    (4100, 16, 16, 128, 128, 3, "4,1,2,1"),      # input and output above 4 GiB
    (2060, 64, 16, 90, 91, 3, "4,1,2,1"),        # the input alone; images that end inside a tile
    (4100, 64, 64, 64, 64, 1, "2,2,1,2"),        # a pointwise layer
    (2050, 16, 48, 128, 128, 5, "4,1,1,1"),      # a window without tiles of its own, from 2 GiB on
])
def test_conv2d_large_tensors(N, Ci, Co, H, W, k, tile):
    """Byte offsets beyond 31 and 32 bits: the gather kernel, against the same images in three batches that the other kernels take."""
    p = k // 2
    args = (Ci, Co, H, W, k, k, 1, (p, p, p, p), 16, 16)
    assert S.small_conv2d_kernel(N, *args) == f"conv16_mfma<{tile}>" and not S.small_conv2d_kernel(N // 3 + 1, *args).startswith("conv16_mfma")
    g = torch.Generator(DEV).manual_seed(N)
    x = torch.rand(N * Ci * H * W, device=DEV, generator=g) * 2 - 1
    w = torch.rand(Co * Ci * k * k, device=DEV, generator=g) * 2 - 1
    per_in, per_out = Ci * H * W, Co * H * W
    out = torch.full((N * per_out + 64,), CANARY, device=DEV)
    S.small_conv2d(x, w, out[:N * per_out], N, *args)
    assert bool((out[N * per_out:] == CANARY).all())
    for lo in range(0, N, N // 3 + 1):
        n = min(N // 3 + 1, N - lo)
        part = torch.empty(n * per_out, device=DEV)
        S.small_conv2d(x[lo * per_in:(lo + n) * per_in], w, part, n, *args)
        # two sums of K products of at most 1, each with at most K roundings of 2^-24 of the largest partial sum
        assert float((out[lo * per_out:(lo + n) * per_out] - part).abs().max()) <= 2 * (Ci * k * k) ** 1.5 * 2.0 ** -24


SPARSE_FILTERS = {  # worst error in 2^-24 of sum |x w|, or None; 2-norm error relative to the result's
    "one": (2.1, 3.5e-8),       # one weight per output: the product's dropped part and the final rounding, 2^-24 each
    "two": (3.1, 4.2e-8),       # two: one more rounding, of the large products' sum
    "box": (None, 8e-8),        # 1/9 under one channel: ten roundings, fewer at full size; with all products in one sum 1.3e-7
    "rectified": (None, 2.6e-7),      # dense weights, inputs >= 0: 3.1e-7 with the fp32 instruction, 3.6e-7 in one sum
}


@pytest.mark.parametrize("kind", sorted(SPARSE_FILTERS))
@pytest.mark.parametrize("N,Ci,Co,H,W,k", [(64, 64, 64, 28, 28, 3), (24, 16, 64, 37, 35, 5)])
def test_conv2d_three_part_products_precision(kind, N, Ci, Co, H, W, k):
    """Filters of few weights, where every rounding of a small product at the size of a large one would show, and rectified
    inputs, whose sums grow all the way."""
    p = k // 2
    assert S.small_conv2d_kernel(N, Ci, Co, H, W, k, k, 1, (p, p, p, p), 16, 16).startswith("conv16_split3")
    rng = np.random.default_rng(8500 + N)
    x = rng.standard_normal((N, Ci, H, W)).astype(np.float32)
    dense = (rng.standard_normal((Co, Ci, k, k)) * np.sqrt(2 / (Ci * k * k))).astype(np.float32)
    w = np.zeros_like(dense)
    if kind == "box":
        w[:, 3] = np.float32(1 / 9)
    elif kind == "rectified":
        w, x = dense, np.maximum(x, 0)
    else:
        w[:, 1, p, p] = dense[:, 1, p, p]
        if kind == "two":
            w[:, Ci - 1, 0, 0] = dense[:, Ci - 1, 0, 0]
    got = run_conv(x, w, 1, (p, p, p, p))
    idx = np.r_[0, 1, N // 2, N - 1]
    xd, wd = torch.from_numpy(x[idx]).double(), torch.from_numpy(w).double()
    ref = torch.nn.functional.conv2d(xd, wd, padding=p).numpy()
    size = torch.nn.functional.conv2d(xd.abs(), wd.abs(), padding=p).numpy()
    err = np.abs(got[idx] - ref)
    worst, rel = SPARSE_FILTERS[kind]
    if worst is not None:
        assert (err <= worst * 2.0 ** -24 * size).all(), (err / np.maximum(size, 1e-30)).max() * 2 ** 24
    assert np.linalg.norm(err) <= rel * np.linalg.norm(ref), np.linalg.norm(err) / np.linalg.norm(ref)


def test_conv2d_three_part_products_infinities():
    """Values without three parts: a workgroup that meets one computes its tile value by value. An infinity and a NaN in the
    input, a filter value that rounds past the largest bf16, and the largest float."""
    N, C, H = 40, 64, 28
    rng = np.random.default_rng(8400)
    x = (rng.random((N, C, H, H), dtype=np.float32) * 2 - 1).astype(np.float32)
    w = (rng.random((C, C, 3, 3), dtype=np.float32) + np.float32(0.5)).astype(np.float32)
    x[3, 5, 10, 11], x[7, 63, 0, 0], x[9, 0, 27, 27] = np.inf, np.nan, np.finfo(np.float32).max
    clean = run_conv(np.nan_to_num(np.where(np.abs(x) > 2, 0, x), nan=0.0), w, 1, (1, 1, 1, 1))
    got = run_conv(x, w, 1, (1, 1, 1, 1))
    ref = O.conv2d(x[[3, 7, 9]], w, 1, (1, 1, 1, 1))
    bad = ~np.isfinite(ref)
    assert np.array_equal(np.isnan(got[[3, 7, 9]]), np.isnan(ref)) and np.array_equal(got[[3, 7, 9]] == np.inf, ref == np.inf)
    assert bad[0].sum() == 9 * C and bad[1].sum() == 4 * C
    ok = np.isfinite(ref) & (np.abs(ref) < 1e6)
    assert np.abs(got[[3, 7, 9]][ok] - ref[ok]).max() <= 576 * 2.0 ** -23 * 1.5
    rest = np.delete(np.arange(N), [3, 7, 9])
    assert np.abs(got[rest] - clean[rest]).max() <= 576 * 2.0 ** -23 * 1.5
    w[17, 3, 1, 1] = np.finfo(np.float32).max          # its bf16 is infinite
    got = run_conv(clean_x := np.nan_to_num(np.where(np.abs(x) > 2, 0, x), nan=0.0), w, 1, (1, 1, 1, 1))
    ref = O.conv2d(clean_x[[0]], w, 1, (1, 1, 1, 1))
    both = np.isfinite(ref)
    assert np.array_equal(np.isfinite(got[[0]]), both)
    # sums of sixteen products, then of these: at most 16 + 36 roundings, each at most 2^-24 of sum |x w|
    size = O.conv2d(np.abs(clean_x[[0]]), np.abs(w), 1, (1, 1, 1, 1))
    err = np.abs(got[[0]][both].astype(np.float64) - ref[both])
    assert (err <= 52 * 2.0 ** -24 * size[both].astype(np.float64)).all()


@pytest.mark.parametrize("case", SPLIT3_CASES)
def test_conv2d_three_part_products_scattered_infinities(case):
    """Tiles with an infinity or a NaN go by the fp32 instruction: strips, ragged ends, windows and padding once more. Outputs whose
    window has none stay as exact as K + 1 roundings allow; in the last run a filter value is infinite too, which a tap in the
    padding must not multiply."""
    N, Ci, Co, H, W, kh, kw, pad = case
    rng = np.random.default_rng(8450 + N)
    x = (rng.random((N, Ci, H, W), dtype=np.float32) * 2 - 1).astype(np.float32)
    w = (rng.random((Co, Ci, kh, kw), dtype=np.float32) * 2 - 1).astype(np.float32)
    idx = np.unique(np.r_[0, 1, N // 2, N - 1])
    x[idx, 3 % Ci, 0, 0], x[idx, Ci - 1, H - 1, W - 2], x[idx, 0, H // 2, W // 2] = np.inf, -np.inf, np.nan
    size = O.conv2d(np.abs(np.nan_to_num(x[idx], nan=0, posinf=0, neginf=0)), np.abs(w), 1, pad)
    for bad_weight in (False, True):
        if bad_weight:
            w[min(5, Co - 1), 0, 0, 0] = np.inf
        got, ref = run_conv(x, w, 1, pad)[idx], O.conv2d(x[idx], w, 1, pad)
        ok = np.isfinite(ref)
        assert ok.mean() > 0.2 and not ok.all()
        assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.array_equal(got[~ok], ref[~ok], equal_nan=True)
        assert (np.abs(got[ok].astype(np.float64) - ref[ok]) <= (Ci * kh * kw + 1) * 2.0 ** -23 * size[ok]).all()


WIDE_CASES = [  # N, Ci, Co, H, W, kh, kw, pad: 256-pixel tiles, a wave 64 x 64, workgroups that walk over tiles
    (60, 96, 48, 27, 33, 3, 3, (1, 1, 1, 1)),        # fewer tiles than compute units; three chunks; three output blocks of four
    (94, 64, 96, 103, 9, 3, 3, (1, 1, 1, 1)),        # two to three tiles a workgroup, which end inside images; six output blocks
    (40, 96, 64, 27, 51, 3, 3, (1, 0, 2, 0)),        # uneven padding: 26 x 51 outputs, the last strip shorter
    (900, 64, 64, 56, 7, 3, 3, (1, 1, 1, 1)),        # narrow images
]


@pytest.mark.parametrize("case", WIDE_CASES)
@pytest.mark.parametrize("scale", [1.0, 1e-36, 1e30])
def test_conv2d_three_part_wide_tiles(case, scale):
    N, Ci, Co, H, W, kh, kw, pad = case
    assert S.small_conv2d_kernel(N, Ci, Co, H, W, kh, kw, 1, pad, 16, 16).startswith("conv16_split3_wide"), case
    test_conv2d_three_part_products(case, scale)


@pytest.mark.parametrize("case", WIDE_CASES)
def test_conv2d_three_part_wide_tiles_scattered_infinities(case):
    N, Ci, Co, H, W, kh, kw, pad = case
    assert S.small_conv2d_kernel(N, Ci, Co, H, W, kh, kw, 1, pad, 16, 16).startswith("conv16_split3_wide"), case
    test_conv2d_three_part_products_scattered_infinities(case)


@pytest.mark.parametrize("kind", sorted(SPARSE_FILTERS))
def test_conv2d_three_part_wide_tiles_precision(kind):
    assert S.small_conv2d_kernel(20, 64, 64, 64, 47, 3, 3, 1, (1, 1, 1, 1), 16, 16) == "conv16_split3_wide<6>"
    test_conv2d_three_part_products_precision(kind, 20, 64, 64, 64, 47, 3)


EIGHT_PRODUCTS = {  # as SPARSE_FILTERS, where the other choice is the fp32 instruction: no more than its errors
    # The final rounding, 1; seven of the small products' sum inside matrix instructions, which round to within a unit of the last place
    # and not to half of one: 7 x 2 x 2^-7 at most, 0.11 (fp32 1.0, 2.53e-8).
    "one": (1.11, 2.6e-8),
    # And the large products' one, 2 by the same, the small ones' twice: 3.25 (2.24 seen; fp32 1.94, 3.1e-8).
    "two": (3.25, 3.0e-8),
    "box": (None, 8e-8),
    "rectified": (None, 2.6e-7),
}


@pytest.mark.parametrize("kind", sorted(EIGHT_PRODUCTS))
@pytest.mark.parametrize("N,Ci,Co,H,W", [(27, 160, 160, 24, 24), (10, 192, 96, 69, 42)])
def test_conv2d_three_part_wide_tiles_precision_of_fp32(kind, N, Ci, Co, H, W, monkeypatch):
    """Layers that the fp32 instruction would compute otherwise keep its precision, whatever the filter."""
    assert S.small_conv2d_kernel(N, Ci, Co, H, W, 3, 3, 1, (1, 1, 1, 1), 16, 16) == "conv16_split3_wide<8>"
    monkeypatch.setitem(SPARSE_FILTERS, kind, EIGHT_PRODUCTS[kind])
    test_conv2d_three_part_products_precision(kind, N, Ci, Co, H, W, 3)


def test_conv_identity_filter_is_exact():
    rng = np.random.default_rng(5)
    x = rng.standard_normal((2, 32, 10, 12)).astype(np.float32)
    w = np.zeros((32, 32, 3, 3), np.float32)
    w[np.arange(32), np.arange(32), 1, 1] = 1
    assert_bits(run_conv(x, w, 1, (1, 1, 1, 1)), x, "delta filter")


def test_dense():
    rng = np.random.default_rng(6)
    for N, Ci, Co in [(7, 64, 10), (1, 256, 2), (33, 64, 12), (130, 128, 128), (3, 16, 16), (5, 6, 3), (1024, 64, 12)]:
        x = rng.standard_normal((N, Ci, 1, 1)).astype(np.float32)
        w = rng.standard_normal((Co, Ci, 1, 1)).astype(np.float32)
        Cib, Cob = _blk(Ci), _blk(Co)
        g = Guarded(N * Co)
        S.small_dense(dev(O.pack(x, Cib)), dev(O.pack_filter(w, Cob, Cib)), g.t, N, Ci, Co, Cib, Cob)
        got = O.unpack(g.check(), (N, Co, 1, 1), Cob)
        assert_close(got, O.dense(x, w), Ci, f"dense {N}x{Ci}->{Co}")


# ------------------------------------------------------------------ depthwise / pooling

DW_CASES = [  # N, C, H, W, k, stride, pad
    (2, 32, 13, 11, 3, 1, (1, 1, 1, 1)),
    (2, 64, 12, 12, 3, 2, (0, 1, 0, 1)),
    (1, 8, 48, 48, 3, 2, (0, 1, 0, 1)),        # 8-channel block
    (3, 128, 3, 3, 3, 2, (1, 1, 1, 1)),
    (2, 64, 25, 5, 3, 1, (1, 1, 1, 1)),
    (1, 16, 9, 9, 5, 1, (2, 2, 2, 2)),         # run-time window
    (2, 3, 10, 10, 3, 1, (1, 1, 1, 1)),        # scalar path
    (2, 256, 7, 7, 3, 1, (1, 1, 1, 1)),
]


@pytest.mark.parametrize("case", DW_CASES)
def test_dwconv2d(case):
    N, C, H, W, k, s, pad = case
    rng = np.random.default_rng(abs(hash(case)) % 2**31)
    x = (rng.random((N, C, H, W), dtype=np.float32) * 2 - 1).astype(np.float32)
    w = (rng.random((C, 1, k, k), dtype=np.float32) * 2 - 1).astype(np.float32)
    Cb = _blk(C)
    ref = O.dwconv2d(x, w, s, pad)
    g = Guarded(ref.size)
    S.small_dwconv2d(dev(O.pack(x, Cb)), dev(O.pack_dw_filter(w, Cb)), g.t, N, C, H, W, k, k, s, pad, Cb)
    assert_close(O.unpack(g.check(), ref.shape, Cb), ref, k * k, f"dw {case}")


DW_LARGE_CASES = [  # N, C, H, W, stride, pad: at least 40 MB of traffic, where the row-staged kernel takes over
    (8, 64, 161, 97, 1, (1, 1, 1, 1)),         # odd image: ragged row tiles, two row tiles of different height
    (6, 128, 120, 120, 2, (0, 1, 0, 1)),       # stride 2
    (700, 64, 25, 5, 1, (1, 1, 1, 1)),         # two whole small images per tile, last group shifted back (N odd / 2)
    (3501, 32, 7, 7, 1, (1, 1, 1, 1)),         # five images per tile, batch not a multiple of five
    (9, 16, 300, 140, 1, (0, 0, 0, 0)),        # rows wider than half a tile: one row per tile; no padding
    (8, 16, 150, 300, 1, (1, 1, 1, 1)),        # rows wider than a tile: too much to stage, the LDS-tiled kernel runs
]


@pytest.mark.parametrize("case", DW_LARGE_CASES)
def test_dwconv2d_large(case):
    N, C, H, W, s, pad = case
    rng = np.random.default_rng(abs(hash(case)) % 2**31)
    x = (rng.random((N, C, H, W), dtype=np.float32) * 2 - 1).astype(np.float32)
    w = (rng.random((C, 1, 3, 3), dtype=np.float32) * 2 - 1).astype(np.float32)
    ref = O.dwconv2d(x, w, s, pad)
    assert (x.size + ref.size) * 4 >= 40 << 20
    g = Guarded(ref.size)
    S.small_dwconv2d(dev(O.pack(x, 16)), dev(O.pack_dw_filter(w, 16)), g.t, N, C, H, W, 3, 3, s, pad, 16)
    assert_close(O.unpack(g.check(), ref.shape, 16), ref, 9, f"dw large {case}")


DW_LANES_CASES = [  # N, C, H, W: 3x3, stride 1, padding 1, 16-channel blocks
    (6, 64, 56, 56),           # four bands of 14 columns; the planes cut into row strips
    (20, 128, 28, 28),         # two bands
    (70, 256, 14, 14),         # one band: lanes 0 and 15 of a row of lanes stay zero
    (300, 512, 7, 7),          # two planes side by side in the 16 lanes
    (3, 16, 5, 5),             # ... an odd number of planes: the last pair has one
    (5, 48, 7, 3),             # ... narrow
    (1, 16, 1, 1),             # one pixel
    (2, 32, 1, 40),            # one row: every output touches the top and the bottom edge; three bands (14, 14, 12)
    (9, 48, 61, 63),           # three channel blocks, five bands (the last of 7 columns), strips of unequal height
    (70, 32, 33, 17),          # two bands, three columns in the second
    (12, 32, 52, 15),          # 15 columns: one more than a band
    (5, 32, 70, 100),          # eight bands, the last of two columns
    (600, 16, 2, 64),          # two rows
    (400, 16, 33, 8),          # eight columns: one plane per row of lanes again
    (64, 64, 56, 56),          # the benchmark row
]


@pytest.mark.parametrize("case", DW_LANES_CASES)
def test_dwconv2d_lane_shift(case):
    """Depthwise 3x3 layers with stride 1 and padding 1 run with the rows in registers and the horizontal neighbours
    taken from the next lanes: bands and their halo lanes, plane pairs, row strips, both image edges, ragged rows.
    The filters are random, so a shift in the wrong direction or a swapped row shows."""
    N, C, H, W = case
    rng = np.random.default_rng(7300 + N + C)
    x = (rng.random((N, C, H, W), dtype=np.float32) * 2 - 1).astype(np.float32)
    w = (rng.random((C, 1, 3, 3), dtype=np.float32) * 2 - 1).astype(np.float32)
    ref = O.dwconv2d(x, w, 1, (1, 1, 1, 1))
    g = Guarded(ref.size)
    S.small_dwconv2d(dev(O.pack(x, 16)), dev(O.pack_dw_filter(w, 16)), g.t, N, C, H, W, 3, 3, 1, (1, 1, 1, 1), 16)
    assert_close(O.unpack(g.check(), ref.shape, 16), ref, 9, f"dw lanes {case}")


POOL_CASES = [  # N, C, H, W, kh, kw, stride, pad
    (2, 32, 13, 11, 3, 3, 2, (0, 0, 0, 0)),
    (1, 16, 56, 56, 3, 3, 2, (0, 0, 0, 0)),
    (2, 48, 9, 9, 3, 3, 1, (1, 1, 1, 1)),
    (2, 16, 8, 8, 2, 2, 2, (0, 0, 0, 0)),
    (3, 64, 8, 8, 8, 8, 1, (0, 0, 0, 0)),      # global
    (3, 256, 2, 2, 2, 2, 1, (0, 0, 0, 0)),     # global
    (5, 64, 25, 5, 25, 5, 1, (0, 0, 0, 0)),    # global
    (2, 8, 6, 6, 6, 6, 1, (0, 0, 0, 0)),       # global, 8-channel block
    (2, 3, 7, 7, 3, 3, 2, (1, 1, 1, 1)),       # scalar path
]


@pytest.mark.parametrize("case", POOL_CASES)
@pytest.mark.parametrize("mode", ["max", "avg"])
def test_pool2d(case, mode):
    N, C, H, W, kh, kw, s, pad = case
    rng = np.random.default_rng(abs(hash(case)) % 2**31)
    x = (rng.random((N, C, H, W), dtype=np.float32) * 2 - 1).astype(np.float32)
    Cb = _blk(C)
    ref = O.pool2d(x, (kh, kw), s, pad, mode)
    g = Guarded(ref.size)
    S.small_pool2d(dev(O.pack(x, Cb)), g.t, N, C, H, W, kh, kw, s, pad, Cb, S.POOL_MAX if mode == "max" else S.POOL_AVG)
    got = O.unpack(g.check(), ref.shape, Cb)
    if mode == "max":
        assert_bits(got, ref, f"maxpool {case}")
    else:
        assert_close(got, ref, kh * kw, f"avgpool {case}")


POOL_LARGE_CASES = [  # N, C, H, W, stride, pad: tens of MB, many workgroups per plane
    (16, 64, 112, 112, 2, (0, 0, 0, 0)),       # the sweep's pooling geometry, smaller batch
    (8, 64, 161, 97, 1, (1, 1, 1, 1)),         # padded: taps outside the image
    (4201, 32, 8, 8, 2, (0, 1, 0, 1)),         # many tiny images
]


@pytest.mark.parametrize("case", POOL_LARGE_CASES)
@pytest.mark.parametrize("mode", ["max", "avg"])
def test_pool2d_large(case, mode):
    N, C, H, W, s, pad = case
    rng = np.random.default_rng(abs(hash(case)) % 2**31)
    x = (rng.random((N, C, H, W), dtype=np.float32) * 2 - 1).astype(np.float32)
    if mode == "max":      # ties between +0 and -0, NaNs, whole windows of NaN
        flat = x.reshape(-1)
        idx = rng.integers(0, flat.size, flat.size // 7)
        flat[idx[0::3]] = 0.0
        flat[idx[1::3]] = -0.0
        flat[idx[2::3]] = np.nan
        x[0, :, :6, :6] = np.nan
        x[-1, :, -5:, :] = -0.0
    ref = O.pool2d(x, (3, 3), s, pad, mode)
    g = Guarded(ref.size)
    S.small_pool2d(dev(O.pack(x, 16)), g.t, N, C, H, W, 3, 3, s, pad, 16, S.POOL_MAX if mode == "max" else S.POOL_AVG)
    got = O.unpack(g.check(), ref.shape, 16)
    if mode == "max":
        assert_bits(got, ref, f"maxpool large {case}")
    else:
        assert_close(got, ref, 9, f"avgpool large {case}")


@pytest.mark.parametrize("shape", [(2, 16, 3, 3), (2, 32, 16, 16), (1, 16, 20, 31), (3, 48, 33, 30), (2, 16, 4, 5), (1, 16, 57, 125),
                                   (2, 16, 31, 15), (1, 32, 16, 17), (7, 80, 14, 14), (4, 256, 56, 56)])
def test_maxpool_3x3_stride_2_by_lane_shifts(shape):
    """The 3x3 / stride 2 / unpadded window on 16-channel blocks: bands of 16 pixels (7 outputs) and strips of 7 output rows, at
    widths of one band, a band and one pixel, many bands, and heights that split into ragged strips; +0 / -0 ties, NaNs and
    whole windows of NaN as the reference scan resolves them."""
    N, C, H, W = shape
    rng = np.random.default_rng(N * 1000 + H * 10 + W)
    x = (rng.random((N, C, H, W), dtype=np.float32) * 2 - 1).astype(np.float32)
    flat = x.reshape(-1)
    idx = rng.integers(0, flat.size, flat.size // 5)
    flat[idx[0::4]] = 0.0
    flat[idx[1::4]] = -0.0
    flat[idx[2::4]] = np.nan
    flat[idx[3::4]] = -np.inf
    x[0, :, :3, :3] = np.nan
    ref = O.pool2d(x, (3, 3), 2, (0, 0, 0, 0), "max")
    g = Guarded(ref.size)
    S.small_pool2d(dev(O.pack(x, 16)), g.t, N, C, H, W, 3, 3, 2, (0, 0, 0, 0), 16, S.POOL_MAX)
    assert_bits(O.unpack(g.check(), ref.shape, 16), ref, f"maxpool 3x3 s2 {shape}")


def test_maxpool_ties_and_nan_bit_exact():
    x = np.zeros((1, 16, 4, 4), np.float32)
    x[0, :, 0, 0], x[0, :, 0, 1] = -0.0, 0.0          # first seen is -0
    x[0, :, 2, 2], x[0, :, 2, 3], x[0, :, 3, 2], x[0, :, 3, 3] = np.nan, -3.0, np.nan, -5.0
    x[0, :, 0, 2], x[0, :, 0, 3], x[0, :, 1, 2], x[0, :, 1, 3] = 0.0, -0.0, -1.0, -2.0
    x[0, :, 1, 0], x[0, :, 1, 1] = -0.0, -0.0
    ref = O.pool2d(x, (2, 2), 2)
    g = Guarded(ref.size)
    S.small_pool2d(dev(O.pack(x, 16)), g.t, 1, 16, 4, 4, 2, 2, 2, (0, 0, 0, 0), 16, S.POOL_MAX)
    assert_bits(O.unpack(g.check(), ref.shape, 16), ref, "maxpool specials")


def test_errors_leave_output_untouched():
    x = dev(np.ones(16 * 64, np.float32))
    g = Guarded(16 * 64)
    with pytest.raises(S.binding.SmallError):
        S.small_conv2d(x, x, g.t, 1, 16, 24, 8, 8, 3, 3, 1, (1, 1, 1, 1), 16, 16)
    with pytest.raises(S.binding.SmallError):
        S.small_pool2d(x, x, 1, 16, 8, 8, 3, 3, 1, (1, 1, 1, 1), 16, S.POOL_MAX)
    assert (g.check() == np.float32(-7.25e37)).all()


def test_matrix_rate_probe_computes_what_it_says():
    """small_probe_mfma: eight accumulators, each `iters` times A x B with A[i][k] = 0.25 + (i & 7) / 1000 and
    B = 0.75, so D[i][j] = iters * 4 * 0.75 * A[i]; a lane holds rows 4q .. 4q+3 and stores the sum over its 32 values."""
    wgs, iters = 3, 5
    g = Guarded(wgs * 256)
    S.small_probe_mfma(g.t, wgs, iters)
    got = g.check().reshape(wgs, 4, 64)
    lane = np.arange(64)
    q = lane // 16
    rows = np.stack([4 * q + r for r in range(4)])                   # rows held by a lane
    ref = (8 * iters * 4 * 0.75 * (0.25 + (rows & 7) / 1000.0).sum(axis=0)).astype(np.float32)
    assert np.allclose(got, ref[None, None, :], rtol=1e-5, atol=0)


def test_matrix_and_vector_probe_computes_what_it_says():
    """small_probe_mfma_valu: four accumulators, each 4 * iters times A x B as above, and valu * iters multiply-adds
    a * b spread over eight registers, with a = 0.25 + (lane & 7) / 1000 and b = 0.75."""
    wgs, iters = 2, 3
    lane = np.arange(64)
    q = lane // 16
    rows = np.stack([4 * q + r for r in range(4)])
    for valu in (0, 32, 64, 96):
        g = Guarded(wgs * 256)
        S.small_probe_mfma_valu(g.t, wgs, iters, valu)
        got = g.check().reshape(wgs, 4, 64)
        ref = 4 * 4 * iters * 4 * 0.75 * (0.25 + (rows & 7) / 1000.0).sum(axis=0) + valu * iters * (0.25 + (lane & 7) / 1000.0) * 0.75
        assert np.allclose(got, ref.astype(np.float32)[None, None, :], rtol=1e-5, atol=0), valu
    with pytest.raises(RuntimeError):
        S.small_probe_mfma_valu(g.t, wgs, iters, 7)


# ------------------------------------------------------------------ seeded random geometries

def _random_geometry(rng, max_hw=34):
    kh, kw = int(rng.choice([1, 1, 3, 3, 3, 2, 5])), int(rng.choice([1, 1, 3, 3, 3, 2, 4]))
    if rng.random() < 0.6:
        kw = kh
    stride = int(rng.choice([1, 1, 1, 2, 2, 3]))
    H, W = int(rng.integers(kh, max_hw)), int(rng.integers(kw, max_hw))
    pad = (int(rng.integers(0, kh)), int(rng.integers(0, kh)), int(rng.integers(0, kw)), int(rng.integers(0, kw)))
    return H, W, kh, kw, stride, pad


@pytest.mark.parametrize("seed", range(48))
def test_conv2d_random_geometries(seed):
    """Channel counts, image sizes, windows, strides and paddings drawn from a seeded generator: whatever kernel the
    dispatcher picks for the geometry has to agree with the definition."""
    rng = np.random.default_rng(9000 + seed)
    Ci = int(rng.choice([1, 3, 8, 16, 16, 32, 48, 64, 128]))
    Co = int(rng.choice([8, 10, 16, 16, 32, 48, 64, 128]))
    H, W, kh, kw, stride, pad = _random_geometry(rng)
    N = int(rng.integers(1, 6)) if seed % 4 else int(rng.integers(20, 70))
    x = (rng.random((N, Ci, H, W), dtype=np.float32) * 2 - 1).astype(np.float32)
    w = (rng.random((Co, Ci, kh, kw), dtype=np.float32) * 2 - 1).astype(np.float32)
    got = run_conv(x, w, stride, pad)
    assert_close(got, O.conv2d(x, w, stride, pad), Ci * kh * kw,
                 f"conv N={N} {Ci}->{Co} {H}x{W} k={kh}x{kw} s={stride} pad={pad}")


@pytest.mark.parametrize("seed", range(32))
def test_window_layers_random_geometries(seed):
    rng = np.random.default_rng(9500 + seed)
    C = int(rng.choice([3, 8, 16, 16, 32, 64, 80]))
    Cb = _blk(C)
    H, W, kh, kw, stride, pad = _random_geometry(rng, 40)
    N = int(rng.integers(1, 5)) if seed % 3 else int(rng.integers(30, 90))
    x = rng.standard_normal((N, C, H, W)).astype(np.float32)
    w = rng.standard_normal((C, 1, kh, kw)).astype(np.float32)
    Ho, Wo = O.out_dim(H, kh, stride, pad[0], pad[1]), O.out_dim(W, kw, stride, pad[2], pad[3])
    xb = dev(O.pack(x, Cb))
    what = f"N={N} C={C} {H}x{W} k={kh}x{kw} s={stride} pad={pad}"
    g = Guarded(N * C * Ho * Wo)
    S.small_dwconv2d(xb, dev(O.pack_dw_filter(w, Cb)), g.t, N, C, H, W, kh, kw, stride, pad, Cb)
    assert_close(O.unpack(g.check(), (N, C, Ho, Wo), Cb), O.dwconv2d(x, w, stride, pad), kh * kw, "dw " + what)
    g = Guarded(N * C * Ho * Wo)
    S.small_pool2d(xb, g.t, N, C, H, W, kh, kw, stride, pad, Cb, S.POOL_MAX)
    assert_bits(O.unpack(g.check(), (N, C, Ho, Wo), Cb), O.pool2d(x, (kh, kw), stride, pad, "max"), "max pool " + what)
    g = Guarded(N * C * Ho * Wo)
    S.small_pool2d(xb, g.t, N, C, H, W, kh, kw, stride, pad, Cb, S.POOL_AVG)
    assert_close(O.unpack(g.check(), (N, C, Ho, Wo), Cb), O.pool2d(x, (kh, kw), stride, pad, "avg"), kh * kw, "avg pool " + what)
