"""The module that takes tensors to the C calls: plain arguments go through, everything else is left to the general path."""
import contextlib
import shutil
import subprocess
import sys

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2512_19849_amd import binding, runner  # noqa: E402


@pytest.fixture(scope="module")
def call():
    binding.load_library()
    from paper_2512_19849_amd import _epcall
    _epcall.set_address_type(binding.Address)
    return _epcall


T8, TK = torch.zeros(8), torch.zeros(4, 2, dtype=torch.int32)


def combine(call, h=0, y=T8, w=T8, dst=TK, T=4, rows=8, out=T8, stream=0):
    return call.ep_combine(h, y, w, dst, T, rows, out, stream)


@pytest.mark.parametrize("change", [{}, dict(y=None), dict(y=binding.Address(64)), dict(rows=2**40), dict(T=-1),
                                    dict(w=torch.nn.Parameter(torch.zeros(8))), dict(out=torch.zeros(0))])
def test_plain_arguments_reach_the_call(call, change):
    assert combine(call, **change) == binding.EP_EINVAL          # (no handle)


@pytest.mark.parametrize("change", [dict(y=8), dict(y=np.zeros(8)), dict(y=torch.zeros(4, 4).t()), dict(y=True), dict(T=4.0),
                                    dict(T=True), dict(T=np.int64(4)), dict(T=2**31), dict(rows=2**63), dict(T=T8),
                                    dict(h=True), dict(h=2**70), dict(stream=object()), dict(dst=TK.to_sparse()),
                                    dict(out=type("Sub", (torch.Tensor,), {})(8))])
def test_anything_else_is_left_alone(call, change):
    assert combine(call, **change) is NotImplemented
    assert call.ep_combine(0, T8, T8, TK, 4, 8, T8) is NotImplemented


def test_batched_tensors_are_left_alone(call):
    seen = []
    torch.vmap(lambda y: (seen.append(combine(call, y=y)), y)[1])(torch.zeros(3, 8))
    assert seen == [NotImplemented]


@pytest.mark.parametrize("src", [0, 2, -1, 3, np.int32(2), True, torch.tensor(1)])
def test_rows(call, src, monkeypatch):
    monkeypatch.setattr(binding, "_fast", call)
    for t in (torch.zeros(3, 5, 2, dtype=torch.int32), torch.zeros(3, 10)[:, :5], torch.zeros(3, 7, dtype=torch.float64)):
        if src.__class__ is int and src == 3:
            with pytest.raises(IndexError):
                runner._row(t, src)
        elif src is True:
            assert runner._row(t, src).shape == t[src].shape
        else:
            assert binding._ptr(runner._row(t, src)) == t[src].data_ptr()
    assert call.row(torch.zeros(()), 0) is NotImplemented and call.row(torch.zeros(0, 3), 0) is NotImplemented


@pytest.fixture
def fresh(monkeypatch):
    """The binding as it is before the first call of a program whose device torch has initialised."""
    import paper_2512_19849_amd as package
    binding.load_library()
    monkeypatch.setattr(binding, "_torch_c", None)
    monkeypatch.setattr(binding, "_fast", binding._General())
    monkeypatch.setattr(binding, "_fast_tried", False, raising=False)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda *a: None)
    monkeypatch.setattr(torch._C, "_cuda_getDevice", lambda: 0, raising=False)
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda device: 0, raising=False)
    monkeypatch.delattr(package, "_epcall", raising=False)
    return monkeypatch


@pytest.mark.parametrize("file", [False, True, "of another torch"])
def test_the_library_is_whole_without_the_module(fresh, call, file, tmp_path):
    if file == "of another torch":
        fresh.setattr(torch, "__version__", "0.0")
    else:
        fresh.setitem(sys.modules, "paper_2512_19849_amd._epcall", None)  # (its import fails)
        fresh.setattr(binding._build, "CALL", str(tmp_path / "_epcall.so"))
        if file:
            (tmp_path / "_epcall.so").write_bytes(b"")
    for first in (True, False):
        with pytest.warns(RuntimeWarning) if file and first else contextlib.nullcontext():
            with pytest.raises(binding.EPError) as e:
                binding.ep_combine(0, T8, T8, TK, 4, 8, T8)
        assert e.value.rc == binding.EP_EINVAL and isinstance(binding._fast, binding._General)


class Stream:
    cuda_stream = 0


@pytest.mark.parametrize("stream", [0, Stream()])
def test_callers_that_pass_a_stream_get_the_direct_calls(fresh, call, stream):
    for ready in (False, True):
        fresh.setattr(torch.cuda, "is_initialized", lambda: ready)
        with pytest.raises(binding.EPError):
            binding.ep_combine(0, T8, T8, TK, 4, 8, T8, stream=stream)
        assert (binding._fast is call) == ready
    assert combine(call, stream=stream) == binding.EP_EINVAL
    assert combine(call, stream=type("Odd", (), {"cuda_stream": "0"})()) is NotImplemented


THROWS = """
import importlib.util, sys, threading, torch
spec = importlib.util.spec_from_file_location("_epcall", sys.argv[1])
call = importlib.util.module_from_spec(spec)
spec.loader.exec_module(call)
t = torch.zeros(4, 2, dtype=torch.int32)
for _ in range(2):
    try:
        print("returned", call.ep_combine(0, t, t, t, 4, 8, t, 0))
    except RuntimeError as e:
        print("raised", e)
worker = threading.Thread(target=print, args=("alive",))
worker.start()
worker.join()
"""


def test_an_exception_out_of_the_library_is_raised(monkeypatch, tmp_path):
    from paper_2512_19849_amd import build
    if not shutil.which("g++"):
        pytest.skip("g++ is not available")
    names = ["layout", "dispatch", "recv_wait", "fp8_unpack", "ht_dispatch", "dedup", "gather_index", "combine_partial"]
    (tmp_path / "lib.cpp").write_text("#include <new>\nextern \"C\" {\nint ep_combine() { throw std::bad_alloc(); }\n" +
                                      "".join(f"int ep_{n}() {{ return 0; }}\n" for n in names) + "}\n")
    subprocess.run(["g++", "-shared", "-fPIC", "-o", str(tmp_path / "libep.so"), str(tmp_path / "lib.cpp")], check=True)
    monkeypatch.setattr(build, "HERE", str(tmp_path))
    monkeypatch.setattr(build, "CALL", str(tmp_path / "_epcall.so"))
    build.build_call()
    r = subprocess.run([sys.executable, "-c", THROWS, build.CALL], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.split("\n")[:3] == ["raised std::bad_alloc"] * 2 + ["alive"], r.stdout + r.stderr
