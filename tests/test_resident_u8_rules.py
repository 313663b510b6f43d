"""What the image-resident quantized runs accept (host arithmetic of resident_u8.hip, no GPU needed)."""
import ctypes as C

import pytest


class Quant(C.Structure):          # QuantParams
    _fields_ = [(n, C.c_int) for n in ("zx", "zw", "zy", "mult", "shift", "lo", "hi", "amax", "mult32")]


class AddQuant(C.Structure):
    _fields_ = [(n, C.c_int) for n in ("za", "zb", "zy", "mult_a", "mult_b", "shift", "lo", "hi")]


class Group(C.Structure):          # RU8Group of small_internal.h
    _fields_ = ([(n, C.c_int) for n in ("kind", "src", "src2", "dst", "Ci", "Co", "Cob", "H", "W", "Ho", "Wo", "kh", "kw", "stride",
                                        "pt", "pl")] +
                [("filt", C.c_void_p), ("sums", C.c_void_p), ("q", Quant), ("qa", AddQuant)])


CONV, DW, ADD, AVG, DENSE = range(5)


@pytest.fixture(scope="module")
def takes():
    from paper_2303_04769_amd import binding
    f = binding.load()["_ZN5small17resident_u8_takesERKNS_8RU8GroupE"]
    f.restype = C.c_bool
    return lambda **kw: f(C.byref(_group(**kw)))


def _group(kind, C_, H=1, W=1, Co=None, k=1, sums=0x1000, filt=0x1000, Cob=16, zx=100):
    g = Group(kind=kind, src=0, src2=0, dst=1, Ci=C_, Co=Co or C_, Cob=Cob, H=H, W=W, Ho=H, Wo=W, kh=k, kw=k, stride=1, pt=k // 2,
              pl=k // 2, filt=filt, sums=sums)
    g.q = Quant(zx, 128, 128, 1 << 20, 30, 0, 255, 1000, 1 << 22)
    return g


def test_units_are_divided_exactly_up_to_the_block_limit(takes):
    """A unit's output block is unit - blocks * (unit ceil(2^20 / blocks) >> 20): exact for every layer that is taken, wrong
    from 1025 blocks on."""
    def exact(blocks):
        inv, groups = -(-(1 << 20) // blocks), -(-(4096 // blocks) // 16)
        return all((u * inv) >> 20 == u // blocks for u in range(groups * blocks))
    assert all(exact(b) for b in range(1, 1025)) and not exact(1025)
    assert takes(kind=DW, C_=16 * 1024) and takes(kind=CONV, C_=16, Co=4096)
    for blocks in (1025, 1057, 2047, 4096):
        assert not takes(kind=DW, C_=16 * blocks), blocks


def test_layers_that_are_taken(takes):
    assert takes(kind=CONV, C_=64, H=8, W=8, k=3) and takes(kind=DW, C_=64, H=25, W=5, k=3)
    assert takes(kind=DENSE, C_=64, Co=12, Cob=12) and takes(kind=ADD, C_=32, H=9, W=9) and takes(kind=AVG, C_=32, H=9, W=9)
    assert not takes(kind=CONV, C_=64, H=8, W=8, k=3, sums=None) and takes(kind=CONV, C_=64, H=8, W=8, k=3, sums=None, zx=128)
    assert not takes(kind=CONV, C_=64, H=8, W=8, k=3, sums=0x1004) and not takes(kind=CONV, C_=64, H=40, W=40, k=3)
    assert not takes(kind=DENSE, C_=64, Co=12, Cob=12, sums=0x1004)


def test_overlaps_are_refused_as_by_the_layers_own_calls():
    """A first layer whose filter or channel sums lie in the buffer it writes, and an output that lies in the workspace: the
    layer's own call refuses them, before anything is launched, and so does the table whose layers would be one launch. (Device
    addresses that are never used: without the overlap the call gets as far as the launch, which has no device here.)"""
    from paper_2303_04769_amd import binding as B
    import torch
    if torch.cuda.is_available():
        pytest.skip("the addresses are not real")
    lib = B.load()
    ws, out, inp, filt, sums = 0x100000, 0x800000, 0x400000, 0xa00000, 0xb00000

    def run(filt0=filt, sums0=sums, out=out):
        t = (B.small_layer_u8 * 3)()
        for k, (src, dst) in enumerate([(-1, 0), (0, 1), (1, -2)]):
            t[k].op, t[k].Ci, t[k].Co, t[k].Cib, t[k].Cob = B._OPS["conv"], 32, 32, 16, 16
            t[k].kh = t[k].kw = t[k].stride = 1
            t[k].src, t[k].dst = src, dst
            t[k].filt, t[k].filt_sums = (filt0, sums0) if k == 0 else (filt + 4096 * k, sums + 4096 * k)
            t[k].q = B.small_quant(100, 128, 128, 1 << 20, 30, 0, 255)
        return lib.small_network_run_u8(t, 3, inp, out, ws, 1 << 16, 4, 32, 5, 5, None)

    assert run() not in (0, 4)
    assert run(filt0=ws + 64) == 4 and run(sums0=ws + 64) == 4 and run(filt0=ws + 4 * 32 * 25 - 16) == 4
    assert run(filt0=ws + 0x8000) not in (0, 4)
