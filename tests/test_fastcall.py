"""The C++ marshalling of the forward calls against the Python one beside it: what it does not take goes to the Python code, with that code's
errors; on the GPU the same statuses, stream and results."""
import ctypes
import importlib.util
import os
import subprocess

import pytest
import torch

import paper_2603_05168_amd.binding as b


def test_built_and_declines_what_it_does_not_know():
    assert b._fastcall is not None
    ws, Y, X = torch.zeros(256, dtype=torch.uint8), torch.zeros(2, 8), torch.zeros(2, 8, dtype=torch.bfloat16)
    rest = (None, None, None, None, 0)
    assert b._fast_linear(X, ws, ws, Y, 2, 4, ws, *rest) is None                # not on a GPU
    assert b._fast_linear(X, 4096, ws, Y, 2, 4, ws, *rest) is None              # an address
    assert b._fast_linear(X, ws, ws, torch.nn.Parameter(Y), 2, 4, ws, *rest) is None
    assert b._fast_linear(X[0], ws, ws, Y, 2, 4, ws, *rest) is None             # one dimension
    assert b._fast_linear(X, ws) is None
    assert b._fast_grouped(b"short", 2, 4, 0, ws) is None
    with pytest.raises(TypeError):
        b.sbn_sparse_ternary_linear(X.float(), ws, ws, Y, 2, 4, ws)
    with pytest.raises(ValueError):
        b.sbn_sparse_ternary_linear(X[0], ws, ws, Y, 2, 4, ws)


def _layer(tokens=5, d_in=512, d_out=96):
    from gpu_util import hip_pack
    import sbn_synth
    packed, gamma = hip_pack(sbn_synth.latent_weight(d_out, d_in, 77), 2, 4)
    X = sbn_synth.activations(tokens, d_in, 78).cuda()
    ws = b.new_workspace(b.sbn_workspace_bytes(b.SBN_OP_LINEAR, tokens, d_out, d_in, 2, 4))
    return X, packed, gamma, ws


@pytest.mark.gpu
def test_same_results_streams_and_errors(monkeypatch):
    X, packed, gamma, ws = _layer()
    out = {}
    for name in ("fast", "python"):
        if name == "python":
            monkeypatch.setattr(b, "_fast_linear", lambda *args: None)
            monkeypatch.setattr(b, "_fast_grouped", lambda *args: None)
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        Y = [torch.full((5, 96), float("nan"), device="cuda") for _ in range(3)]
        bias = torch.arange(96, dtype=torch.float32, device="cuda")
        torch.cuda.synchronize()
        with torch.cuda.stream(side):
            assert b._fastcall.stream() == side.cuda_stream
            b.sbn_sparse_ternary_linear(X, packed, gamma, Y[0], 2, 4, ws)
            b.LinearGroup([X, X], [packed] * 2, [gamma] * 2, Y[1:], 2, 4, b.new_workspace(2 * ws.numel())).run()
        assert b._fastcall.stream() == torch.cuda.current_stream().cuda_stream
        torch.cuda.synchronize()
        xq, sx = torch.zeros(5, 512, dtype=torch.int8, device="cuda"), torch.zeros(5, device="cuda")
        Yb, Yq = torch.zeros(5, 96, device="cuda"), torch.zeros(5, 96, device="cuda")
        b.sbn_sparse_ternary_linear(X, packed, gamma, Yb, 2, 4, ws, bias=bias, xq_out=xq, sx_out=sx)
        b.sbn_sparse_ternary_linear(None, packed, gamma, Yq, 2, 4, ws, xq_out=xq, sx_out=sx)
        b.sbn_sparse_ternary_linear(X, packed.data_ptr(), gamma, Yb[:, :], 2, 4, ws, bias=bias.data_ptr())
        torch.cuda.synchronize()
        assert torch.equal(Y[0], Y[1]) and torch.equal(Y[0], Y[2]) and torch.equal(Y[0], Yq)
        errors = []
        for call in (lambda: b.sbn_sparse_ternary_linear(X, packed, gamma, Yb, 9, 4, ws),
                     lambda: b.sbn_sparse_ternary_linear(X, packed, gamma, Yb, 2, 4, ws[:256]),
                     lambda: b.sbn_sparse_ternary_linear(X, packed[4:], gamma, Yb, 2, 4, ws),
                     lambda: b.sbn_sparse_ternary_linear(X, None, gamma, Yb, 2, 4, ws),
                     lambda: b.LinearGroup([X], [packed], [gamma], [Yb], 2, 4, ws[:256]).run()):
            with pytest.raises(b.SbnError) as e:
                call()
            errors.append((e.value.status, str(e.value)))
        out[name] = [y.cpu() for y in Y + [Yb, Yq]] + errors
    assert all(torch.equal(a, c) if torch.is_tensor(a) else a == c for a, c in zip(out["fast"], out["python"]))


@pytest.mark.gpu
@pytest.mark.parametrize("fast", [True, False])
def test_group_runs_on_the_arrays_it_has_now(monkeypatch, fast):
    # attributes set after construction count, on both paths; the arrays that they replace are not looked at again
    if not fast:
        monkeypatch.setattr(b, "_fast_grouped", lambda *args: None)
    X, packed, gamma, ws = _layer()
    Y = [torch.full((5, 96), float("nan"), device="cuda") for _ in range(4)]
    group = b.LinearGroup([X, X], [packed] * 2, [gamma] * 2, Y[:2], 2, 4, b.new_workspace(2 * ws.numel()))
    group.run()
    torch.cuda.synchronize()
    want = Y[0].clone()
    for y in Y:
        y.fill_(float("nan"))
    group.Y = b._ptr_array(Y[2:])
    group.run()
    torch.cuda.synchronize()
    assert torch.equal(Y[2], want) and torch.equal(Y[3], want) and Y[0].isnan().all() and Y[1].isnan().all()
    group.count, group.tokens = 1, b._i64_array([3, 3])
    for y in Y:
        y.fill_(float("nan"))
    group.run()
    torch.cuda.synchronize()
    assert torch.equal(Y[2][:3], want[:3]) and Y[2][3:].isnan().all() and Y[3].isnan().all()
    group.Y[0] = Y[0].data_ptr()          # an entry written in place
    group.run()
    torch.cuda.synchronize()
    assert torch.equal(Y[0][:3], want[:3])


def test_group_arrays_of_another_kind_are_left_to_python():
    arrays = {"X": b._ptr_array([64]), "tokens": b._i64_array([1])}
    assert b._fastcall.array_of_pointers(arrays["X"], 1) and b._fastcall.array_of_integers(arrays["tokens"], 1)
    for other in (arrays["tokens"], b"12345678", [64], torch.zeros(1, dtype=torch.int64).numpy(), ctypes.pointer(ctypes.c_void_p(64)), None):
        assert not b._fastcall.array_of_pointers(other, 1)
    for other in (arrays["X"], (ctypes.c_int32 * 2)(), torch.zeros(1, dtype=torch.int64).numpy(), ctypes.pointer(ctypes.c_int64(1)), None):
        assert not b._fastcall.array_of_integers(other, 1)
    assert not b._fastcall.array_of_pointers(arrays["X"], 2)      # shorter than the count


def test_exceptions_of_a_call_reach_python_with_its_lock_held(tmp_path):
    source = tmp_path / "throws.cpp"
    source.write_text("""#include <new>
#include <stdexcept>
extern "C" int fine() { return -3; }
extern "C" int no_memory() { throw std::bad_alloc(); }
extern "C" int message() { throw std::runtime_error("as it says"); }
extern "C" int anything() { throw 7; }
""")
    subprocess.run(["g++", "-shared", "-fPIC", "-o", tmp_path / "throws.so", source], check=True)
    lib = ctypes.CDLL(str(tmp_path / "throws.so"))
    address = lambda f: ctypes.cast(f, ctypes.c_void_p).value   # noqa: E731
    assert b._fastcall.call(address(lib.fine)) == -3
    for f, error, text in ((lib.no_memory, MemoryError, None), (lib.message, RuntimeError, "as it says"), (lib.anything, RuntimeError, "unknown")):
        with pytest.raises(error, match=text):
            b._fastcall.call(address(f))
    assert b._fastcall.call(address(lib.fine)) == -3


def _build_script():
    spec = importlib.util.spec_from_file_location("sbn_build_script", os.path.join(os.path.dirname(b.__file__), "build.py"))
    module = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(module)
    return module


def test_package_without_the_marshalling(tmp_path, monkeypatch, capsys):
    # a compiler that is missing or fails is a warning, and no library of an earlier build is left in its place
    script = _build_script()
    monkeypatch.setattr(script, "FASTCALL_LIB", str(tmp_path / "_fastcall.so"))
    for compiler in ("no-such-compiler", "false"):
        (tmp_path / "_fastcall.so").write_bytes(b"old")
        assert script.build_fastcall(compiler) is False
        assert not (tmp_path / "_fastcall.so").exists() and "was not built" in capsys.readouterr().err
    assert b._load_fastcall(str(tmp_path / "_fastcall.so")) is None
    assert not script.fastcall_is_current()


def test_marshalling_built_for_another_torch_is_not_used(monkeypatch):
    script, path = _build_script(), b._fastcall.__file__
    assert b._fastcall.torch_version == torch.__version__ and script.fastcall_is_current() and b._load_fastcall(path) is not None
    monkeypatch.setattr(torch, "__version__", "0.0")
    assert not script.fastcall_is_current() and b._load_fastcall(path) is None
