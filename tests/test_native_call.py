"""The extension module that marshals calls into the library: what it does not take is left to ctypes, whose errors a caller
sees, and nothing is left behind by a call that fails on the way."""
import ctypes
import os
import shutil
import subprocess
import sys
import sysconfig

import pytest
import torch

from paper_2509_21354_amd import binding as kb
from paper_2509_21354_amd import build as kvev_build


def _args(**kw):
    kb.lib()
    t = torch.zeros(64)
    a = dict(shape=kb.make_shape(L=1, B=1, H=1, d=64, T=8, T_cap=8, C=4, N_cap=2, W=4, d_sum=32, d_g=64, dtype=kb.F32, H_kv=0),
             Q=t, Tq=1, K=t, V=t, Kbar=t, Vbar=t, idx=t.int(), count=t.int(), k_cap=1, O=t, ws=None, causal=0)
    a.update(kw)
    return a


def _call(**kw):
    return kb._native.gated_attention(*_args(**kw).values())


@pytest.mark.skipif(torch.cuda.is_available(), reason="the GPU is not initialised here")
def test_plain_calls_wait_for_the_gpu():
    assert _call() is None                   # (ctypes' way then says that there is no GPU)
    with pytest.raises((RuntimeError, AssertionError)):
        kb.kvev_gated_attention(**_args())


@pytest.mark.parametrize("kw", [dict(shape=None), dict(shape=ctypes.c_int(0)), dict(Tq=1.0), dict(Tq=2 ** 40), dict(k_cap="1"), dict(Q=3),
                                dict(ws=kb.RowsFrom(torch.zeros(4, 4), 1, 4)), dict(causal=None)])
def test_other_arguments_are_left_to_ctypes(kw):
    assert _call(**kw) is None


def test_wrong_number_of_arguments_is_not_taken():
    assert kb._native.gated_attention() is None
    assert kb._native.retain(*range(40)) is None


def test_strided_tensors_are_refused():
    with pytest.raises(AssertionError, match="contiguous"):
        _call(V=torch.zeros(4, 4).t())
    with pytest.raises(AssertionError, match="contiguous"):
        kb.kvev_gated_attention(**_args(V=torch.zeros(4, 4).t()))


def test_errors_of_a_tensor_reach_the_caller_and_nothing_is_held():
    class Odd(torch.Tensor):
        def data_ptr(self):
            raise ValueError("no address")

    a = _args(K=torch.zeros(4).as_subclass(Odd))
    before = sys.getrefcount(a["shape"]), sys.getrefcount(a["K"])
    for _ in range(3):
        with pytest.raises(ValueError, match="no address"):
            kb._native.gated_attention(*a.values())
    assert (sys.getrefcount(a["shape"]), sys.getrefcount(a["K"])) == before


CHILD = """
import torch
from paper_2509_21354_amd import binding as kb
torch.cuda._initialized = True                 # what a process forked from one that used the GPU finds
torch.cuda.is_initialized = lambda: False      # what torch answers there
kb.lib()
t = torch.zeros(64)
sh = kb.make_shape(L=1, B=1, H=1, d=64, T=8, T_cap=8, C=4, N_cap=2, W=4, d_sum=32, d_g=64, dtype=kb.F32, H_kv=0)
assert kb._native.gated_attention(sh, t, 1, t, t, t, t, t.int(), t.int(), 1, t, None, 0) is None
"""


def test_torch_is_asked_whether_the_gpu_is_up():
    """A forked child inherits torch's flag, not the GPU: torch says no there, and ctypes' way raises torch's error."""
    r = subprocess.run([sys.executable, "-c", CHILD], capture_output=True, text=True, cwd=os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
    assert r.returncode == 0, r.stderr[-2000:]


@pytest.mark.gpu
def test_a_forked_child_is_refused():
    """... before anything reaches the GPU (the child makes no call of it)."""
    rows = torch.zeros(8, 64)
    a = {k: v.cuda() if isinstance(v, torch.Tensor) else v for k, v in _args(K=rows, V=rows, Kbar=rows, Vbar=rows).items()}
    kb.kvev_gated_attention(**a)
    torch.cuda.synchronize()
    pid = os.fork()
    if pid == 0:
        code = 1
        try:
            kb.kvev_gated_attention(**a)
        except RuntimeError as e:
            code = 0 if "fork" in str(e) else 2
        finally:
            os._exit(code)
    assert os.waitpid(pid, 0)[1] == 0


WITHOUT = """
import ctypes, os, sys, warnings
warnings.simplefilter("error" if {quiet} else "always")
from paper_2509_21354_amd import binding as kb
assert os.path.dirname(kb.__file__) == {where!r}
{between}
sh = kb.make_shape(L=1, B=1, H=1, d=64, T=8, T_cap=8, C=4, N_cap=2, W=4, d_sum=32, d_g=64, dtype=kb.BF16, H_kv=0)
assert kb.workspace_bytes(kb.OP_LSTM_GATE, sh, 2) > 0
print("native" if kb._native else "ctypes")
"""


def _package_without_extension(tmp_path):
    where = tmp_path / "paper_2509_21354_amd"
    where.mkdir()
    for name in ("__init__.py", "binding.py", "build.py", "synth.py", "cost_model.py", "libkvev.so"):
        shutil.copy(os.path.join(os.path.dirname(kb.__file__), name), where / name)
    return where


def _child(where, between="", quiet=True):
    code = WITHOUT.format(where=str(where), between=between, quiet=quiet)
    r = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, cwd=where.parent)
    assert r.returncode == 0, r.stderr[-2000:]
    return r.stdout.strip(), r.stderr


def test_the_library_works_without_the_extension(tmp_path):
    assert _child(_package_without_extension(tmp_path))[0] == "ctypes"


def test_an_extension_built_after_the_import_is_taken(tmp_path):
    where = _package_without_extension(tmp_path)
    assert _child(where, f"import shutil; shutil.copy({kvev_build.NATIVE_PATH!r}, {str(where)!r})")[0] == "native"


def test_an_extension_that_does_not_load_is_named(tmp_path):
    where = _package_without_extension(tmp_path)
    (where / os.path.basename(kvev_build.NATIVE_PATH)).write_bytes(b"no shared object")
    out, err = _child(where, quiet=False)
    assert out == "ctypes" and "does not load" in err


def test_build_goes_on_without_a_host_compiler(tmp_path, monkeypatch, capsys):
    stale = tmp_path / os.path.basename(kvev_build.NATIVE_PATH)
    stale.write_bytes(b"old")
    monkeypatch.setattr(kvev_build, "NATIVE_PATH", str(stale))
    monkeypatch.setattr(kvev_build, "CXX", str(tmp_path / "no-such-compiler"))
    kvev_build._build_native(True, 0.0)
    assert not stale.exists() and "ctypes" in capsys.readouterr().err


def test_the_extension_is_named_for_its_python():
    assert kvev_build.NATIVE_PATH.endswith(sysconfig.get_config_var("EXT_SUFFIX"))
