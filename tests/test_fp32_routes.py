"""Which kernel fp32 group convolutions take (host arithmetic of conv.hip, no GPU needed)."""
import ctypes as C

import pytest


@pytest.fixture(scope="module")
def group_tile():
    """The tile of the matrix-core kernels that takes a group convolution (N, Ci, F_C, S_C, K, H, W, k, stride, pad), or -1."""
    from paper_2303_04769_amd import binding
    f = binding.load()["_ZN5small20group_conv_same_tileERKNS_9LayerGeomEiii"]

    def call(N, Ci, F_C, S_C, K, H, W, k, s, pad, Cib=16, Cob=16):
        Ho, Wo, G = (H + pad[0] + pad[1] - k) // s + 1, (W + pad[2] + pad[3] - k) // s + 1, (Ci - F_C) // S_C + 1
        return f((C.c_int * 14)(N, H, W, Ho, Wo, Ci, G * K, Cib, Cob, k, k, s, pad[0], pad[2]), F_C, S_C, K)
    return call


def test_group_convolutions_on_the_matrix_cores(group_tile):
    """Whatever the size: the other choice is a lane per output (64 -> 64 channels in two groups, stride 2, 8 x 8, one image 52 us
    there, 6.0 here)."""
    from test_gpu_table2 import GROUP_CASES
    for N, Ci, F_C, S_C, K, H, W, k, s, pad, Cib, F_Cb, Cob in GROUP_CASES:
        whole = Cib == F_Cb == Cob == 16 and F_C % 16 == S_C % 16 == K % 16 == 0
        assert (group_tile(N, Ci, F_C, S_C, K, H, W, k, s, pad, Cib, Cob) >= 0) == whole, (N, Ci, F_C, S_C, K, H, W)
    for N in (1, 16, 4096):
        for W in (2, 7, 8, 56):
            assert group_tile(N, 64, 32, 32, 32, 8, W, 3, 2, (1, 1, 1, 1)) >= 0
    # rows whose first pixel has a tap 0 inside the image and whose last one a tap 2; stride 3
    assert group_tile(1, 64, 32, 32, 32, 8, 7, 3, 2, (0, 0, 0, 0)) < 0
    assert group_tile(1, 64, 32, 32, 32, 8, 9, 3, 3, (1, 1, 1, 1)) < 0
