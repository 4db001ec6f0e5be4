"""The native marshalling of the binding (CPU): its table against the C ABI's
argument lists, and the calls it leaves to the checks in Python."""
import ctypes
import os
import re

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
