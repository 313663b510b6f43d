"""Which kernel quantized convolutions with windows take (host arithmetic of conv_u8_tile.hip, no GPU needed)."""
import ctypes as C

import pytest


@pytest.fixture(scope="module")
def tiles():
    """True where conv_u8_tile takes the layer (N, Ci, Co, H, W, kh, kw, stride, pad), its filter sums given."""
    from paper_2303_04769_amd import binding
    f = binding.load()["_ZN5small21conv_u8_tile_eligibleERKNS_9LayerGeomERKNS_11QuantParamsEPKiPKv"]
    f.restype = C.c_bool

    def call(N, Ci, Co, H, W, kh, kw, s, pad, sums=0x1000, out=0x1000, zx=100, amax=1000, zw=128):
        Ho, Wo = (H + pad[0] + pad[1] - kh) // s + 1, (W + pad[2] + pad[3] - kw) // s + 1
        geom = (C.c_int * 14)(N, H, W, Ho, Wo, Ci, Co, 16, 16, kh, kw, s, pad[0], pad[2])
        quant = (C.c_int * 9)(zx, zw, 128, 1 << 20, 30, 0, 255, amax, 1 << 22)          # QuantParams
        return f(geom, quant, C.c_void_p(sums), C.c_void_p(out))
    return call


@pytest.fixture(scope="module")
def tile_form():
    """(tile, streamed) of a layer that conv_u8_tile takes."""
    from paper_2303_04769_amd import binding

    class Form(C.Structure):
        _fields_ = [("tile", C.c_int), ("stream", C.c_bool)]
    f = binding.load()["_ZN5small17conv_u8_tile_formERKNS_9LayerGeomE"]
    f.restype = Form

    def call(N, Ci, Co, H, W, kh, kw, s, pad, *_):
        Ho, Wo = (H + pad[0] + pad[1] - kh) // s + 1, (W + pad[2] + pad[3] - kw) // s + 1
        form = f((C.c_int * 14)(N, H, W, Ho, Wo, Ci, Co, 16, 16, kh, kw, s, pad[0], pad[2]))
        return form.tile, form.stream, N * Co * Ho * Wo
    return call


P1 = (1, 1, 1, 1)


def test_tile_kernel_where_it_is_faster(tiles):
    """Both sides of the line, each measured (us, register kernels / tiles)."""
    for layer in [(64, 128, 128, 28, 28, 3, 3, 1, P1),        # 22.4 / 17.1
                  (64, 64, 64, 56, 56, 3, 3, 1, P1),          # 26 / 22
                  (5, 240, 64, 57, 57, 3, 3, 1, P1)]:         # 28.0 / 14.4
        assert tiles(*layer), layer
    for layer in [(1, 16, 16, 32, 32, 3, 3, 1, P1),                       # nine chunks
                  (64, 512, 512, 7, 7, 3, 3, 1, P1),                      # 24.5 / 27.0
                  (102, 272, 128, 14, 14, 2, 2, 1, (0, 0, 0, 0)),         # 19.3 / 35.3
                  (12, 512, 48, 35, 35, 1, 3, 1, (0, 0, 0, 0)),           # 9.2 / 13.4
                  (112, 128, 16, 53, 34, 2, 2, 2, (0, 0, 0, 0))]:         # 6.6 / 11.9
        assert not tiles(*layer), layer


def test_tile_kernel_on_short_reductions(tiles):
    """Large layers of nine or eighteen chunks, those of the parity test, and layers on the other side of each line."""
    from test_gpu_u8 import SHORT_TILE_CASES
    for N, Ci, Co, H, W, s, zx, zw in SHORT_TILE_CASES:
        assert tiles(N, Ci, Co, H, W, 3, 3, s, P1, zx=zx, zw=zw), (N, Ci, Co)
    assert not tiles(490, 32, 32, 28, 28, 3, 3, 1, P1, zw=131)          # groups of two, sums of the codes: 19.1 / 17.8 us on 106 43x104
    for N, Ci, Co, H, W, s in [(60, 32, 80, 58, 13, 1), (80, 32, 208, 27, 28, 2), (80, 16, 144, 29, 22, 1), (60, 32, 256, 29, 28, 1),
                               (480, 32, 32, 28, 28, 1), (490, 32, 32, 56, 56, 2), (650, 32, 16, 27, 27, 1), (700, 16, 32, 27, 27, 1)]:
        assert not tiles(N, Ci, Co, H, W, 3, 3, s, P1), (N, Ci, Co)
    assert not tiles(90, 16, 144, 29, 22, 3, 1, 1, (1, 1, 0, 0)) and not tiles(66, 32, 80, 58, 13, 3, 3, 1, P1, sums=None)


def test_tile_kernel_conditions(tiles):
    layer = (64, 128, 128, 28, 28, 3, 3, 1, P1)
    assert not tiles(*layer, out=0x1008) and not tiles(*layer, amax=0) and not tiles(*layer, sums=None)
    assert tiles(*layer, sums=None, zx=128)


def test_parity_cases_reach_the_tile_kernel(tiles):
    from test_gpu_u8 import TILE_CASES, TILE_CASES_ELSEWHERE
    for case in TILE_CASES:
        assert tiles(*case[:9]) == (case not in TILE_CASES_ELSEWHERE), case


def test_streamed_tiles(tile_form, tiles):
    """Outputs of 4 MB and more are streamed, but by tiles 5 and 9, which write words of a block; the parity test of streamed
    outputs reaches every one that does."""
    import random
    from test_gpu_u8 import STREAMED_TILE_CASES
    rng = random.Random(3)
    for _ in range(4000):
        H, W, k = rng.randrange(1, 60), rng.randrange(1, 60), rng.choice([2, 3, 5])
        layer = (int(2 ** rng.uniform(0, 13)), 16 * rng.randrange(1, 20), 16 * rng.randrange(1, 20), H + k, W + k, k, k, 1, (k // 2,) * 4)
        tile, stream, out_bytes = tile_form(*layer)
        assert stream == (tile not in (-1, 5, 9) and out_bytes >= 4 << 20), (layer, tile)
    assert sorted(STREAMED_TILE_CASES) == [0, 1, 2, 3, 4, 6, 7, 8]
    for tile, (N, Ci, Co, H, W, k) in STREAMED_TILE_CASES.items():
        layer = (N, Ci, Co, H, W, k, k, 1, (k // 2,) * 4)
        assert tiles(*layer) and tile_form(*layer)[:2] == (tile, True), tile


def test_parity_cases_reach_the_pointwise_walk(tiles, tile_form):
    """Every row of the walk's own test, the row of the test of scales, and the streamed rows of scales above a half."""
    from paper_2303_04769_amd import binding
    from test_gpu_u8 import POINTWISE_AT_A_HALF, STREAMED_AT_A_HALF, test_conv_pointwise_walk, test_conv_pointwise_walk_streamed
    f = binding.load()["_ZN5small19conv_u8_pw_eligibleERKNS_9LayerGeomERKNS_11QuantParamsEPKiPKv"]
    f.restype = C.c_bool
    quant = (C.c_int * 9)(100, 128, 128, (1 << 30) + 1, 31, 0, 255, 1025, -1)

    def walk(N, Ci, Co, H, W, s=1):
        geom = (C.c_int * 14)(N, H, W, (H - 1) // s + 1, (W - 1) // s + 1, Ci, Co, 16, 16, 1, 1, s, 0, 0)
        return f(geom, quant, C.c_void_p(0x1000), C.c_void_p(0x1000))
    rows = [r[:6] for r in test_conv_pointwise_walk.pytestmark[0].args[1]] + [r[:5] for r in test_conv_pointwise_walk_streamed.pytestmark[0].args[1]]
    for row in rows + [POINTWISE_AT_A_HALF]:
        assert walk(*row), row
    assert not walk(9, *POINTWISE_AT_A_HALF[1:])
    for N, Ci, Co, H, W, k, zx, zw in STREAMED_AT_A_HALF:
        layer = (N, Ci, Co, H, W, k, k, 1, (k // 2,) * 4)
        assert walk(N, Ci, Co, H, W) and N * Co * H * W >= 10 << 20 if k == 1 else tiles(*layer) and tile_form(*layer)[1], layer


@pytest.fixture(scope="module")
def dw_form():
    """(waves, rows of a strip, strips side by side) of a depthwise 3x3 layer of stride 1 padded by one."""
    from paper_2303_04769_amd import binding

    class Form(C.Structure):
        _fields_ = [("waves", C.c_long), ("rows", C.c_int), ("fold", C.c_bool)]
    f = binding.load()["_ZN5small14dw_dpp_u8_formERKNS_9LayerGeomE"]
    f.restype = Form

    def call(N, Ci, H, W):
        form = f((C.c_int * 14)(N, H, W, H, W, Ci, Ci, 16, 16, 3, 3, 1, 1, 1))
        return form.waves, form.rows, form.fold
    return call


@pytest.mark.parametrize("W", range(1, 8))
def test_narrow_planes_of_few_images_fill_their_lanes(dw_form, W):
    """The depthwise kernel puts several planes of up to seven pixels a row side by side on a wave's lanes, of consecutive images or,
    of one or a few images, strips of the same plane: at least two fifths of the lanes have a pixel, whatever the number of images."""
    for N in range(1, 40):
        for Ci in (16, 512, 4096, 16384):
            H = (1 << 25) // (N * Ci * W) // 9 * 9 + 9                     # (strips of 9 rows: layers that fill the chip)
            waves = dw_form(N, Ci, H, W)[0]
            assert 0.4 * waves * (16 // W if W <= 5 else 2) <= N * (Ci // 16) * (H // 9) + Ci // 16, (N, Ci, H)


def test_parity_cases_reach_the_depthwise_forms(dw_form):
    from test_gpu_u8 import FOLDED_DW_CASES
    forms = [dw_form(*shape) + (shape[3] <= 5,) for shape in FOLDED_DW_CASES]
    assert all(f[2] for f in forms)
    assert {(f[1], f[3]) for f in forms} == {(rows, narrow) for rows in (3, 5, 7, 9) for narrow in (False, True)}
    for shape in [(17, 16, 3100, 1), (9, 512, 300, 1), (2, 1024, 300, 6), (1, 512, 300, 8), (1, 128, 40, 4), (1, 32, 3, 1)]:
        assert not dw_form(*shape)[2], shape
