"""The native calls of the binding and those in Python that stand in for them: as many arguments as the entry points take, the errors of
the Python check, nothing left of a handle that was closed, and a binding that works without the native ones.  No GPU: no call here gets
past the library's own argument checks."""
import ctypes
import os
import subprocess

import pytest
import torch

from paper_2411_10003_amd import binding
from paper_2411_10003_amd import build as hip_build

if not (os.path.exists(binding.LIB_PATH) and os.path.exists(binding.PYCALL_PATH)):
    hip_build.build()

ENTRIES = ["moe_gate_topk", "moe_expert_counts", "moe_dispatch", "moe_dispatch_after_counts", "moe_expert_ffn_fwd", "moe_combine",
           "moe_combine_bwd", "moe_expert_ffn_bwd", "moe_expert_ffn_bwd_acc", "moe_dispatch_bwd", "moe_gate_bwd", "moe_gate_bwd_params",
           "moe_input_grad"]


def _handle():
    return binding.Handle(T=8, d=64, h=64, E=8, k=1, P=4, self_dest=0, G=2, dtype="bf16", act="swiglu", renorm=0, alloc_workspace=False)


KINDS = ["native", "python"]


def _type(kind):
    native = binding._call_type()
    assert native is not binding.PythonCall
    return native if kind == "native" else binding.PythonCall


def _call(hd, name, handle=0, kind="native"):
    entry = ctypes.cast(getattr(hd.lib, name), ctypes.c_void_p).value
    return _type(kind)(entry, (handle, *hd._spec(name), "int"), binding._ptr)


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("name", ENTRIES)
def test_arguments_of_every_entry(name, kind):
    hd = _handle()
    spec = hd._spec(name)
    assert len(spec) + 2 == len(getattr(hd.lib, name).argtypes)
    # no handle: the library refuses the call (MOE_ERR_NULL)
    assert _call(hd, name, kind=kind)(*(0 if a == "int" else None for a in spec), 0) == -1
    # tensors that are not on a device, by name, as the Python check says it
    first = [a for a in spec if a != "int"][0]
    with pytest.raises(ValueError, match=f"{first[2]}: need a contiguous device tensor"):
        _call(hd, name, kind=kind)(*(0 if a == "int" else torch.zeros(4) for a in spec), 0)
    with pytest.raises(TypeError):
        _call(hd, name, kind=kind)(0)
    with pytest.raises(AttributeError):
        _call(hd, name, kind=kind)(*(0 if a == "int" else "no tensor" for a in spec), 0)
    with pytest.raises(TypeError):
        _call(hd, name, kind=kind)(*(None for _ in spec), None)


@pytest.mark.parametrize("kind", KINDS)
def test_the_check_decides_what_is_not_plain(kind):
    """What the native check does not know is asked of the Python check, with the entry's own dtype, size and name."""
    hd, asked = _handle(), []
    entry = ctypes.cast(hd.lib.moe_gate_bwd, ctypes.c_void_p).value

    def check(t, dtype, numel, name):
        asked.append((dtype, numel, name))
        return None
    call = _type(kind)(entry, (0, *hd._spec("moe_gate_bwd"), "int"), check)
    meta = torch.zeros(64, device="meta")
    assert call(meta, meta.t(), torch.zeros(0), None, 0) == -1
    assert asked == [(torch.float32, 8, "dw"), (torch.float32, 64, "logits"), (torch.int32, 8, "idx")]


def test_a_closed_handle_leaves_no_call():
    hd = _handle()
    hd._calls["moe_gate_bwd"] = _call(hd, "moe_gate_bwd", hd._h.value)
    hd.close()
    assert hd._calls == {} and not hd._h


@pytest.mark.parametrize("there", [None, b"not a library"])
def test_without_the_native_calls(monkeypatch, tmp_path, there):
    path = tmp_path / "_pycall.so"
    if there is not None:
        path.write_bytes(there)
    monkeypatch.setattr(binding, "PYCALL_PATH", str(path))
    monkeypatch.setattr(binding, "_call_class", None)
    monkeypatch.setattr(binding, "_stream", lambda: 0)
    hd = _handle()
    with pytest.raises(binding.MoeError, match="moe_gate_bwd: status -1"):
        hd.gate_bwd(None, None, None, None)
    with pytest.raises(ValueError, match="dw: need a contiguous device tensor"):
        hd.gate_bwd(*[torch.zeros(64)] * 4)
    assert isinstance(hd._calls["moe_gate_bwd"], binding.PythonCall)


@pytest.mark.parametrize("compiler", ["absent", "fails"])
def test_build_without_the_native_calls(monkeypatch, tmp_path, capsys, compiler):
    old = tmp_path / "_pycall.so"
    old.write_bytes(b"of other sources")

    def run(cmd, **kw):
        if compiler == "absent":
            raise FileNotFoundError(cmd[0])
        return subprocess.CompletedProcess(cmd, 1, "", "Python.h: No such file or directory")
    monkeypatch.setattr(hip_build, "PYCALL", str(old))
    monkeypatch.setattr(hip_build.subprocess, "run", run)
    hip_build._pycall()
    assert not old.exists() and "native calls not built" in capsys.readouterr().err
