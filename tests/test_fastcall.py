"""The extension in front of the ctypes binding: takes the plain calls, leaves everything else, refuses what ctypes' path refuses."""
import inspect
import runpy
import sysconfig

import numpy as np
import pytest
import torch

import paper_2303_04769_amd as S
from paper_2303_04769_amd import binding as B

Q = B.small_quant(128, 131, 128, 1 << 21, 31, 0, 255)
F, U, I = torch.float32, torch.uint8, torch.int32
CONV = (2, 16, 32, 5, 7, 3, 3, 1, (1, 1, 1, 1), 16, 16)
DW = (2, 16, 5, 7, 3, 3, 1, (1, 1, 1, 1), 16)
DENSE = (3, 32, 16, 16, 16)
N_IN = 2 * 16 * 5 * 7
# name: tensors (type, elements; the last one of the data is the result), the other arguments, place of the result
CALLS = {
    "pack": ([(F, N_IN), (F, N_IN)], (2, 16, 5, 7, 16), 1),
    "unpack": ([(F, N_IN), (F, N_IN)], (2, 16, 5, 7, 16), 1),
    "pack_u8": ([(U, N_IN), (U, N_IN)], (2, 16, 5, 7, 16), 1),
    "unpack_u8": ([(U, N_IN), (U, N_IN)], (2, 16, 5, 7, 16), 1),
    "conv2d": ([(F, N_IN), (F, 32 * 16 * 9), (F, 2 * N_IN)], CONV, 2),
    "conv2d_u8": ([(U, N_IN), (U, 32 * 16 * 9), (U, 2 * N_IN)], CONV + (Q, (I, 32)), 2),
    "dwconv2d": ([(F, N_IN), (F, 16 * 9), (F, N_IN)], DW, 2),
    "dwconv2d_u8": ([(U, N_IN), (U, 16 * 9), (U, N_IN)], DW + (Q,), 2),
    "pool2d": ([(F, N_IN), (F, N_IN)], DW + (S.POOL_MAX,), 1),
    "pool2d_u8": ([(U, N_IN), (U, N_IN)], DW + (S.POOL_AVG,), 1),
    "relu": ([(F, N_IN), (F, N_IN)], (N_IN,), 1),
    "relu_u8": ([(U, N_IN), (U, N_IN)], (N_IN, 128), 1),
    "add": ([(F, N_IN), (F, N_IN), (F, N_IN)], (N_IN,), 2),
    "dense": ([(F, 96), (F, 512), (F, 48)], DENSE, 2),
    "dense_u8": ([(U, 96), (U, 512), (U, 48)], DENSE + (Q, (I, 16)), 2),
}


def _tensor(spec, device, seed):
    g = torch.Generator().manual_seed(seed)
    t = torch.randn(spec[1], generator=g) if spec[0] == F else torch.randint(0, 256, (spec[1],), generator=g).to(spec[0])
    return t.to(device)


def _arguments(name, device):
    tensors, rest, out = CALLS[name]
    args = [_tensor(s, device, k) for k, s in enumerate(tensors)]
    args += [_tensor(r, device, 9) if isinstance(r, tuple) and r and isinstance(r[0], torch.dtype) else r for r in rest]
    return args, out


def _forms(name, args):
    """The same call in forms that are left to ctypes."""
    ints = [k for k, a in enumerate(args) if type(a) is int]
    yield "a number of another type", [np.int64(a) if k == ints[-1] else a for k, a in enumerate(args)]
    for k, a in enumerate(args):
        if isinstance(a, tuple):
            yield "a padding in a list", [list(a) if j == k else b for j, b in enumerate(args)]
            yield "a padding of five", [a + (1,) if j == k else b for j, b in enumerate(args)]
        if isinstance(a, B.small_quant):
            yield "a record of another type", [object() if j == k else b for j, b in enumerate(args)]
    yield "a tensor of a subclass", [args[0].as_subclass(type("T", (torch.Tensor,), {}))] + args[1:]


@pytest.mark.parametrize("name", sorted(CALLS))
def test_only_plain_calls_are_taken(name):
    """Without a GPU: tensors in host memory are refused as ever; a call in another form, with a stream or with an argument
    too few is not looked at."""
    args, _ = _arguments(name, "cpu")
    fast = getattr(B._fast(), name)
    with pytest.raises(TypeError, match="contiguous .* CUDA tensor"):
        fast(*args, None)
    with pytest.raises(TypeError, match="contiguous .* CUDA tensor"):
        getattr(S, "small_" + name)(*args)
    assert fast(*args, object()) is None and fast(*args) is None and fast(*args, None, None) is None
    for what, other in _forms(name, args):
        assert fast(*other, None) is None, what


@pytest.mark.parametrize("why", ["no compiler", "a file that does not load"])
def test_calls_go_through_ctypes_where_there_is_no_extension(monkeypatch, tmp_path, why):
    """Every call gets as far as ctypes' own look at the tensors, here in host memory; the extension is looked for once."""
    from paper_2303_04769_amd import build
    tries = []

    def no_compiler(*args, **kwargs):
        tries.append(args)
        raise FileNotFoundError(2, "No such file or directory", "g++")
    monkeypatch.setattr(build, "FASTCALL", str(tmp_path / "_fastcall.so"))
    monkeypatch.setattr(B, "_fastcall", None)
    monkeypatch.setattr(build.subprocess, "run", no_compiler)
    if why != "no compiler":
        (tmp_path / "_fastcall.so").write_bytes(b"not a shared object")
    for name in sorted(CALLS):
        args, _ = _arguments(name, "cpu")
        assert getattr(B._fast(), name)(*args, None) is None
        with pytest.raises(TypeError, match="contiguous .* CUDA tensor"):
            getattr(S, "small_" + name)(*args)
    assert len(tries) == (why == "no compiler")


def test_a_call_with_a_stream_goes_straight_to_ctypes(monkeypatch):
    class Untouched:
        def __getattr__(self, name):
            raise AssertionError(name)
    monkeypatch.setattr(B, "_fastcall", Untouched())
    for name in sorted(CALLS):
        args, _ = _arguments(name, "cpu")
        with pytest.raises(TypeError, match="contiguous .* CUDA tensor"):
            getattr(S, "small_" + name)(*args, stream=object())


def test_a_file_is_for_one_python_and_one_torch(monkeypatch):
    """The extension reads tensors by torch's headers: one built for another torch or Python has another name and is not loaded."""
    from paper_2303_04769_amd import build
    path = lambda: runpy.run_path(build.__file__)["FASTCALL"]
    assert path() == build.FASTCALL == B._fast().__file__
    monkeypatch.setattr(torch, "__version__", "2.9.1+rocm6.4")
    other = path()
    monkeypatch.undo()
    monkeypatch.setattr(sysconfig, "get_config_var", lambda name: "cpython-312-x86_64-linux-gnu")
    assert len({build.FASTCALL, other, path()}) == 3


@pytest.mark.parametrize("fails", [False, True])
def test_no_half_written_file_is_in_place(monkeypatch, tmp_path, fails):
    """The compiler's output takes its place when it is whole; an earlier file stays until then, and for good if the build fails."""
    from paper_2303_04769_amd import build
    target = tmp_path / "_fastcall.so"
    target.write_text("earlier")

    def compiler(cmd, **kwargs):
        out = cmd[cmd.index("-o") + 1]
        with open(out, "w") as f:
            f.write("half")
            f.flush()
            assert target.read_text() == "earlier"
            f.write(" and half")
        return build.subprocess.CompletedProcess(cmd, int(fails), "an error" if fails else "")
    monkeypatch.setattr(build, "FASTCALL", str(target))
    monkeypatch.setattr(build.subprocess, "run", compiler)
    if fails:
        with pytest.raises(RuntimeError, match="an error"):
            build.build_fastcall(force=True)
    else:
        build.build_fastcall(force=True)
    assert target.read_text() == ("earlier" if fails else "half and half")
    assert [p.name for p in tmp_path.iterdir()] == ["_fastcall.so"]


@pytest.mark.gpu
@pytest.mark.parametrize("name", sorted(CALLS))
def test_both_routes_agree(name):
    """The extension, the ctypes path (a stream given) and keywords: the same bytes; on a side stream that is still to write the
    call's input, the call waits for it; a type or stride it does not take is refused; an error of the library has the same code on
    both routes."""
    args, out = _arguments(name, "cuda:0")
    call = getattr(S, "small_" + name)
    want = None
    for route in ("extension", "ctypes", "keywords") + 4 * ("side",):      # (a stream may share the default one's hardware queue)
        args[out] = torch.zeros_like(args[out])
        if route == "extension":
            assert getattr(B._fast(), name)(*args, None) == 0
        elif route == "ctypes":
            call(*args, stream=torch.cuda.current_stream())
        elif route == "keywords":
            call(**dict(zip(inspect.signature(call).parameters, args)))
        else:
            data, side = args[0].clone(), torch.cuda.Stream()
            args[0].zero_()
            torch.cuda.synchronize()
            with torch.cuda.stream(side):
                torch.cuda._sleep(10_000_000)            # some milliseconds: a call on another stream reads zeros
                args[0].copy_(data)
                call(*args)
        torch.cuda.synchronize()
        got = args[out].cpu()
        want = got if want is None else want
        assert torch.equal(got, want) and got.float().abs().sum() > 0, route
    wrong = list(args)
    wrong[0] = torch.stack([args[0], args[0]], 1)[:, 0]
    for bad in (wrong[0], args[0].double(), args[0].cpu()):
        with pytest.raises(TypeError, match="contiguous .* CUDA tensor"):
            call(*([bad] + args[1:]))
    codes = []
    for kw in ({}, {"stream": torch.cuda.current_stream()}):
        with pytest.raises(S.SmallError) as e:
            call(*([None] + args[1:]), **kw)
        codes.append(e.value.code)
    assert codes[0] == codes[1]
