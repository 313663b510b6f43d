"""Which kernel quantized convolutions with windows take (host arithmetic of conv_u8_tile.hip, no GPU needed)."""
import ctypes as C

import pytest


@pytest.fixture(scope="module")
def tiles():
    """True where conv_u8_tile takes the layer (N, Ci, Co, H, W, kh, kw, stride, pad), its filter sums given."""
    from paper_2303_04769_amd import binding
    f = binding.load()["_ZN5small21conv_u8_tile_eligibleERKNS_9LayerGeomERKNS_11QuantParamsEPKiPKv"]
    f.restype = C.c_bool

    def call(N, Ci, Co, H, W, kh, kw, s, pad, sums=0x1000, out=0x1000, zx=100, amax=1000):
        Ho, Wo = (H + pad[0] + pad[1] - kh) // s + 1, (W + pad[2] + pad[3] - kw) // s + 1
        geom = (C.c_int * 14)(N, H, W, Ho, Wo, Ci, Co, 16, 16, kh, kw, s, pad[0], pad[2])
        quant = (C.c_int * 9)(zx, 128, 128, 1 << 20, 30, 0, 255, amax, 1 << 22)          # QuantParams
        return f(geom, quant, C.c_void_p(sums), C.c_void_p(out))
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


def test_tile_kernel_conditions(tiles):
    layer = (64, 128, 128, 28, 28, 3, 3, 1, P1)
    assert not tiles(*layer, out=0x1008) and not tiles(*layer, amax=0) and not tiles(*layer, sums=None)
    assert tiles(*layer, sums=None, zx=128)


def test_parity_cases_reach_the_tile_kernel(tiles):
    from test_gpu_u8 import TILE_CASES, TILE_CASES_ELSEWHERE
    for case in TILE_CASES:
        assert tiles(*case[:9]) == (case not in TILE_CASES_ELSEWHERE), case
