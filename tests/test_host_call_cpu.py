"""The native marshalling of the binding (CPU): its table against the C ABI's
argument lists, and the calls it leaves to the checks in Python."""
import ctypes
import os
import re
import subprocess
import sys

import pytest
import torch

import paper_2609_34325_amd as dora

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def kinds():
    src = open(os.path.join(ROOT, "paper_2609_34325_amd", "csrc", "host_call.cpp")).read()
    return re.findall(r'\{"(\w+)",\s*\[\]\(void\* fn, const Arg\* a\) \{\s*return at_address\((\w+), fn\)\(([^;]*)\);', src)


def test_table_matches_the_abi():
    dora.load_library()
    table = kinds()
    assert [name for _, name, _ in table] == [name for name, _ in dora._ENTRIES]
    want = {ctypes.c_void_p: "FILAfilas", ctypes.c_int32: "n", ctypes.c_int64: "n", ctypes.c_size_t: "n",
            ctypes.c_int: "n", ctypes.c_float: "e"}
    letter = {torch.float32: "f", torch.int32: "i", torch.int64: "l", None: "a"}
    for (ks, name, body), (_, spec) in zip(table, dora._ENTRIES):
        types = getattr(dora._lib, name).argtypes
        assert len(ks) == len(types) == len(spec)
        assert [int(i) for i in re.findall(r"a\[(\d+)\]", body)] == list(range(len(ks)))   # each argument once, in order
        for k, t, s in zip(ks, types, spec):
            assert k in want[t], (name, k, t)
            assert (s is None) == (k in "nes")
            if s is not None:
                assert k.lower() == letter[s[1]], (name, s)
                assert k.isupper() or s[0] in dora._OPTIONAL


def test_left_to_python():
    lib = dora.load_library()
    i = dora._INDEX["dora_actor_gate"]
    cpu = torch.zeros(4)
    call = dora._native_call
    assert call(i, lib.addresses[i], 1) is NotImplemented                                   # argument count
    assert call(i, lib.addresses[i], cpu, None, 4, 5, 3, cpu, cpu, cpu, cpu, 0) is NotImplemented   # not on the GPU
    assert call(i, lib.addresses[i], None, None, 4, 5, 3, None, None, None, None, 0) is NotImplemented
    assert call(i, lib.addresses[i], "x", None, 4, 5, 3, cpu, cpu, cpu, cpu, 0) is NotImplemented
    with pytest.raises(ValueError):
        call(99, lib.addresses[i])
    with pytest.raises(ValueError, match="p_gate must be on the GPU"):
        dora._call("dora_actor_gate", 0, cpu, None, 4, 5, 3, cpu, cpu, cpu, cpu)
    with pytest.raises(TypeError, match="p_gate must be a torch tensor"):
        dora._call("dora_actor_gate", 0, None, None, 4, 5, 3, cpu, cpu, cpu, cpu)


def test_built():
    """The native marshalling itself is what the other tests run through."""
    dora.load_library()
    assert dora._native_call is not None and dora._native_call is not dora._leave_to_ctypes


def test_library_loads_without_the_native_marshalling():
    """Not built, or built for another Python or torch: calls go through ctypes."""
    code = """
import sys, warnings
sys.modules["paper_2609_34325_amd._host_call"] = None
import torch, paper_2609_34325_amd as dora
with warnings.catch_warnings(record=True) as seen:
    warnings.simplefilter("always")
    lib = dora.load_library()
assert [w for w in seen if "ctypes" in str(w.message)]
i = dora._INDEX["dora_actor_gate"]
assert dora._native_call(i, lib.addresses[i], 1) is NotImplemented
assert dora.dora_status_string(0) == "DORA_OK"
try:
    dora._call("dora_actor_gate", 0, torch.zeros(4), None, 4, 5, 3, *[torch.zeros(4)] * 4)
except ValueError as e:
    assert str(e) == "p_gate must be on the GPU"
else:
    raise AssertionError
"""
    res = subprocess.run([sys.executable, "-c", code], cwd=ROOT, capture_output=True, text=True, timeout=300)
    assert res.returncode == 0, res.stderr


@pytest.mark.parametrize("cxx", ["false", "/no/such/compiler"])
def test_build_without_a_host_compiler(tmp_path, monkeypatch, cxx):
    """The library needs hipcc only; an older marshalling does not stay behind."""
    from paper_2609_34325_amd import build
    host = tmp_path / "_host_call.so"
    host.write_bytes(b"old")
    monkeypatch.setattr(build, "HOST_LIB", str(host))
    monkeypatch.setenv("CXX", cxx)
    with pytest.warns(UserWarning, match="ctypes"):
        build._build_host(False)
    assert not list(tmp_path.iterdir())


def test_arguments_are_checked_before_the_stream():
    """Without a GPU a CPU tensor is what the error names, not the missing device."""
    code = """
import torch, paper_2609_34325_amd as dora
st, scores, keep = torch.zeros(1, dtype=torch.int32), torch.zeros(2, 5), torch.ones(2, dtype=torch.int32)
for call, name in ((lambda: dora.dora_select_pack(scores, keep, torch.zeros(2, 5, 8), cap_rows=2, dev_status=st), "scores"),
                   (lambda: dora.dora_actor_gate(torch.zeros(2), 1, 5, dev_status=st), "p_gate"),
                   (lambda: dora.dora_varlen_attn_plan(torch.zeros(3, dtype=torch.int32), 1, 5, 5, scores, st), "cu_seqlens")):
    try:
        call()
    except ValueError as e:
        assert str(e) == name + " must be on the GPU", e
    else:
        raise AssertionError(name)
assert not torch.cuda.is_initialized()
"""
    env = dict(os.environ, HIP_VISIBLE_DEVICES="", CUDA_VISIBLE_DEVICES="")
    res = subprocess.run([sys.executable, "-c", code], cwd=ROOT, env=env, capture_output=True, text=True, timeout=300)
    assert res.returncode == 0, res.stderr
