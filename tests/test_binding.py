"""The compiled binding (binding/native.cpp) against the Python functions that it stands in front of: the same results for what it
answers, and everything else left to them, so that the same calls raise the same errors; and what takes its place where it
does not fit the torch or the Python that run."""
import ctypes
import importlib.util
import math
import os
import subprocess
import types

import numpy as np
import pytest
import torch

import synth_inputs as si


@pytest.fixture(scope="module")
def cm():
    import paper_2506_03275_amd as cm
    cm.load()
    return cm


def _calls(dev):
    """Arguments of every function that the binding has, small and valid."""
    B, H, N, E, c, D, F, k = 1, 2, 200, 64, 128, 128, 64, 33
    g = si.generator(51, dev)
    r = lambda *shape: si.randn_bf16(shape, g)   # noqa: E731
    q, kk, v, x, w1, w2 = r(B, H, N, E), r(B, H, N, E), r(B, H, N, E), r(B, N, D), r(F, D), r(F, D)
    f32 = lambda *shape: torch.zeros(shape, dtype=torch.float32, device=dev)   # noqa: E731
    i32 = lambda *shape: torch.zeros(shape, dtype=torch.int32, device=dev)     # noqa: E731
    u8 = lambda n: torch.zeros(n, dtype=torch.uint8, device=dev)               # noqa: E731
    idx = torch.arange(k, dtype=torch.int32, device=dev).expand(B, H, 2, k).contiguous()
    counts = torch.full((B, H, 2), k, dtype=torch.int32, device=dev)
    midx, mcounts = idx[:, 0].contiguous(), counts[:, 0].contiguous()
    scale = 1 / math.sqrt(E)
    scores = torch.arange(5 * 104, dtype=torch.float32, device=dev).view(5, 104).sin()
    ones = f32(B, H, N) + 1
    return dict(
        voxel_reorder=[x, torch.empty_like(x), i32(N), None, 4, 2, 7, 14, 0, 2, 4, 4, False],
        topk_cols=[scores[:, :101], scores.flip(0)[:, :101], 7, i32(5, 8), i32(5)],
        attn_sparse_delta=[q, kk, v, idx, counts, r(B, H, N, E), torch.empty_like(q), c, scale, -1.0],
        attn_dense=[q, kk, v, torch.empty_like(q), f32(B, H, 2, N), c, scale, u8(B * H * N * 8)],
        attn_dense_colsum_stale=[q, kk, v, torch.empty_like(q), ones, ones * 50, f32(B, H, 2, N), c, scale, f32(B, H, N), f32(B, H, N)],
        mlp_tile_mean_preact=[x, w1, f32(B, 2, F), c, u8(1 << 20)],
        mlp_sparse_delta=[x, w1, r(F), w2, midx, mcounts, r(B, F, N), r(B, N, D), c, 1, u8(1 << 20)],
        mlp_dense=[x, w1, r(F), w2, r(D), r(B, N, D), r(B, F, N), c, 0])


NAMES = list(_calls("cpu"))


def _outcome(cm, fast, name, args):
    """What a call raises, or the tensors that it was given, as they are behind it."""
    args = [a.clone(memory_format=torch.preserve_format) if type(a) is torch.Tensor and a._base is None else a for a in args]
    before, cm._fast = cm._fast, fast
    try:
        getattr(cm, name)(*args)
    except Exception as e:   # noqa: BLE001
        return type(e).__name__, str(e)
    finally:
        cm._fast = before
    return [a for a in args if isinstance(a, torch.Tensor)]


def _wrong(args):
    """The same arguments with one of them spoiled, each in the ways that a caller may get it wrong."""
    for i, a in enumerate(args):
        if isinstance(a, torch.Tensor):
            spoiled = [a.double(), a[..., :0], a[0], np.zeros(3), 3, None, a.float() if a.dtype != torch.float32 else a.to(torch.bfloat16)]
            spoiled += [torch.cat([a, a], -1)[..., ::2], torch.cat([a, a]), torch.cat([a, a])[::2], a.unsqueeze(0), a.unsqueeze(-1), a.transpose(0, -1)]
            spoiled += [torch.cat([a, a], -1)[..., :a.shape[-1]], a.to("meta"), torch.nn.Parameter(a, requires_grad=False)]
        elif a is None:
            spoiled = ["x", 0]
        else:
            spoiled = [str(a), 2 ** 40 if isinstance(a, int) else math.nan, 2 ** 64 + 7, None, -1, 0.5, True, torch.tensor(1)]
        for s in spoiled:
            yield i, args[:i] + [s] + args[i + 1:]


@pytest.fixture(scope="module")
def on_the_cpu(cm, tmp_path_factory):
    """Both sides with their one question for the GPU turned into one for the CPU, over functions that write down what they are
    given: what a call does, as ('called', arguments), or ('raised', type, text), or None for one that the binding leaves."""
    from paper_2506_03275_amd import build
    at = tmp_path_factory.mktemp("binding")
    text = open(build.NATIVE_SRC).read()
    assert text.count("is_cuda()") == 2
    (at / "native.cpp").write_text(text.replace("is_cuda()", "is_cpu()").replace('"../../include/chipmunk.h"', f'"{os.path.abspath(build.HEADER)}"'))
    swap = {"-O2": "-O0", build.NATIVE_SRC: str(at / "native.cpp"), build.NATIVE: str(at / "native.so")}
    subprocess.run([swap.get(word, word) for word in build._native_command()], check=True, capture_output=True)
    spec = importlib.util.spec_from_file_location("on_the_cpu._native", str(at / "native.so"))
    native = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(native)
    python = types.ModuleType("paper_2506_03275_amd")
    python.__package__, python.__path__, python.__file__ = cm.__package__, cm.__path__, cm.__file__
    text = open(cm.__file__).read()
    assert text.count(".is_cuda") == 3
    exec(compile(text.replace(".is_cuda", ".is_cpu"), "on_the_cpu", "exec"), python.__dict__)
    seen, functions = [], {}

    def recorder(symbol):
        argtypes, restype = cm._SIGNATURES[symbol]
        return ctypes.CFUNCTYPE(restype, *argtypes)(lambda *args: seen.append([str(a) for a in args]) or 0)   # (a NaN is a NaN)
    for name in NAMES:
        functions["chipmunk_" + name] = recorder("chipmunk_" + name)
    native.bind({n: ctypes.cast(f, ctypes.c_void_p).value for n, f in functions.items()}, lambda: 3, lambda device: 70 + device)
    python._lib = types.SimpleNamespace(**functions)
    python._current_device, python._raw_stream = lambda: 3, lambda device: 70 + device

    def outcome(side, name, args):
        seen.clear()
        try:
            answer = getattr(native if side == "native" else python, name)(*args)
        except Exception as e:   # noqa: BLE001
            assert not seen
            return "raised", type(e).__name__, str(e)
        assert len(seen) == (0 if side == "native" and answer is None else 1)
        return ("called", seen[0]) if seen else None
    return outcome


@pytest.mark.parametrize("name", NAMES)
def test_the_binding_calls_what_the_python_functions_call(on_the_cpu, name):
    """What the binding answers it hands to the library as the Python function does, argument for argument; so whatever that one
    refuses, or takes another way, the binding has left alone."""
    args = _calls("cpu")[name]
    optional = {"voxel_reorder": (2, 3), "topk_cols": (1,), "attn_sparse_delta": (4, 5), "attn_dense": (4, 7), "mlp_sparse_delta": (2, 10),
                "attn_dense_colsum_stale": (9, 10), "mlp_tile_mean_preact": (4,), "mlp_dense": (2, 4)}
    for plain in [args] + [args[:i] + [None] + args[i + 1:] for i in optional[name]]:
        called = on_the_cpu("native", name, plain)
        assert called and called[0] == "called" and called == on_the_cpu("python", name, plain)
        assert called[1][-1] == "73"   # the current device's stream
        refused = 0
        for i, bad in _wrong(plain):
            answer, expected = on_the_cpu("native", name, bad), on_the_cpu("python", name, bad)
            assert answer is None or answer == expected, (i, bad[i])
            refused += expected[0] == "raised"
        assert refused >= 4 * len(args)


@pytest.mark.parametrize("name", NAMES)
def test_what_is_wrong_raises_what_it_raised(cm, name):
    """As built, on the CPU, every call is refused; which error it is must not hang on the binding, whose answer is always None."""
    native = cm._fast
    assert native.__name__.endswith("_native")
    args = _calls("cpu")[name]
    assert getattr(native, name)(*args) is None and getattr(native, name)(*args[:-1]) is None and getattr(native, name)() is None
    for i, bad in _wrong(args):
        assert getattr(native, name)(*bad) is None, i
        got = _outcome(cm, native, name, bad)
        assert isinstance(got, tuple) and got == _outcome(cm, cm._Python(), name, bad), i


@pytest.mark.gpu
@pytest.mark.parametrize("name", NAMES)
def test_the_binding_does_what_the_python_functions_do(cm, name):
    native = cm._fast
    args = _calls("cuda")[name]
    assert getattr(native, name)(*[a.clone(memory_format=torch.preserve_format) if type(a) is torch.Tensor and a._base is None else a for a in args]) == 0
    got, want = _outcome(cm, native, name, args), _outcome(cm, cm._Python(), name, args)
    assert isinstance(got, list) and all(torch.equal(a.view(torch.uint8), b.view(torch.uint8)) if a.is_contiguous() else torch.equal(a, b)
                                         for a, b in zip(got, want))
    optional = {"voxel_reorder": (2,), "topk_cols": (1,), "attn_dense": (4,), "mlp_sparse_delta": (2,), "mlp_dense": (2, 4)}
    for i in optional.get(name, ()):
        less = args[:i] + [None] + args[i + 1:]
        got, want = _outcome(cm, native, name, less), _outcome(cm, cm._Python(), name, less)
        assert isinstance(got, list) and all(torch.equal(a, b) for a, b in zip(got, want))
    side = torch.cuda.Stream()   # on the caller's stream, whichever it is
    with torch.cuda.stream(side):
        assert cm._raw_stream(torch.cuda.current_device()) == side.cuda_stream
        again = _outcome(cm, native, name, args)
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(again, _outcome(cm, cm._Python(), name, args)))


@pytest.mark.parametrize("other", ["torch", "revision", "python", "header", "no header"])
def test_a_binding_for_another_torch_python_or_header_is_left_alone(cm, other, monkeypatch, tmp_path):
    """Its code holds the layout of torch's tensors and Python's objects, and the C functions' arguments.  Another torch would often
    load it all the same, because the few functions that it asks for by name are there in most."""
    from paper_2506_03275_amd import build
    lib = cm.load()
    assert build.native_fits() and cm._bind(lib).__name__.endswith("_native")
    if other == "torch":
        monkeypatch.setattr(torch, "__version__", torch.__version__ + ".1")
    elif other == "revision":
        monkeypatch.setattr(torch.version, "git_version", "0" * 40)
    elif other == "python":
        real = build.sysconfig.get_config_var
        monkeypatch.setattr(build.sysconfig, "get_config_var", lambda name: "cpython-399" if name == "SOABI" else real(name))
    elif other == "no header":   # the package alone, without the tree around it
        monkeypatch.setattr(build, "HEADER", str(tmp_path / "none.h"))
    else:
        header = tmp_path / "chipmunk.h"
        header.write_bytes(open(build.HEADER, "rb").read() + b"\n")
        monkeypatch.setattr(build, "HEADER", str(header))
    assert not build.native_fits() and build.is_stale()
    with pytest.warns(RuntimeWarning, match="compiled binding"):
        assert isinstance(cm._bind(lib), cm._Python)


def test_the_library_does_not_need_the_compiled_binding(cm, monkeypatch, tmp_path):
    """The Python functions do every call: a machine with the library and no host compiler loads it as it is."""
    from paper_2506_03275_amd import build
    monkeypatch.setattr(build, "NATIVE", str(tmp_path / "none.so"))
    monkeypatch.setattr(build, "build", lambda verbose=False: pytest.fail("built anew"))
    monkeypatch.setattr(cm, "_lib", None)
    monkeypatch.setattr(cm, "_fast", cm._fast)
    with pytest.warns(RuntimeWarning, match="compiled binding"):
        assert cm.load().chipmunk_status_string(0) == b"ok"
    assert isinstance(cm._fast, cm._Python)
    args = _calls("cpu")["mlp_dense"]
    with pytest.raises(ValueError, match="must live on the GPU"):
        cm.mlp_dense(*args)


@pytest.mark.parametrize("compiler", ["/nonexistent/c++", "false"])
def test_a_build_without_a_host_compiler_gives_the_library(monkeypatch, tmp_path, capfd, compiler):
    """And takes away the binding of an earlier build, whose functions need not be the library's any more."""
    from paper_2506_03275_amd import build
    (tmp_path / "one.hip").write_text('extern "C" int one() { return 1; }\n')
    for name, value in (("CSRC", str(tmp_path)), ("LIB", str(tmp_path / "lib.so")), ("NATIVE", str(tmp_path / "native.so")),
                        ("PROBE_SRC", str(tmp_path / "one.hip")), ("PROBE_LIB", str(tmp_path / "probe.so"))):
        monkeypatch.setattr(build, name, value)
    (tmp_path / "native.so").write_text("of an earlier build")
    monkeypatch.setenv("CXX", compiler)
    assert build.build() == str(tmp_path / "lib.so")
    assert ctypes.CDLL(str(tmp_path / "lib.so")).one() == 1
    assert not (tmp_path / "native.so").exists() and "binding" in capfd.readouterr().err
