"""GPU checks of the binding's two ways into the library: the native marshalling
and ctypes give the same results, and an exception behind an entry point's
address becomes an error of the one call."""
import ctypes

import pytest
import torch

from gpu_util import to_host_bits

pytestmark = pytest.mark.gpu


def pass_through(dora):
    """Select/pack with a plan, attention and FLOP accounting: all outputs."""
    g = torch.Generator(device="cuda").manual_seed(5)
    B, N, H = 3, 50, 2
    scores = torch.randn(B, N, device="cuda", generator=g)
    tokens = torch.randn(B, N, H * 64, device="cuda", generator=g).bfloat16()
    keep = torch.tensor([50, 17, 1], dtype=torch.int32, device="cuda")
    total, ws, st = 68, dora.new_workspace(B, H, N), dora.new_status()
    idx, cu, packed, _ = dora.dora_select_pack_plan(scores, keep, tokens, H, N, total, ws, cap_rows=total, dev_status=st)
    q, k, v = (torch.randn(total, H, 64, device="cuda", generator=g).bfloat16() for _ in range(3))
    out = dora.dora_varlen_attn_execute(q, k, v, cu, N, ws, dev_status=st)
    counts = torch.full((3, B), N, dtype=torch.int32, device="cuda")
    flops, sums, _ = dora.dora_trajectory_flops(counts, d=H * 64, N0=N - 1, patch=16, M=10, dev_status=st)
    torch.cuda.synchronize()
    assert int(st.item()) == 0
    return [to_host_bits(t) for t in (idx, cu, packed, out, flops, sums)]


def test_ctypes_gives_the_same(gpu, monkeypatch):
    native = pass_through(gpu)
    monkeypatch.setattr(gpu, "_native_call", gpu._leave_to_ctypes)
    for a, b in zip(native, pass_through(gpu)):
        assert (a == b).all()


def test_exception_behind_an_entry_point(gpu):
    """The address of a function that throws std::bad_alloc in an entry point's place."""
    throws = ctypes.cast(ctypes.CDLL("libstdc++.so.6")._ZSt17__throw_bad_allocv, ctypes.c_void_p).value
    i = gpu._INDEX["dora_actor_gate"]
    p, n = torch.zeros(4, device="cuda"), torch.zeros(4, dtype=torch.int32, device="cuda")
    for _ in range(3):
        with pytest.raises(RuntimeError, match="threw"):
            gpu._native_call(i, throws, p, None, 4, 5, 3, n, n, n, n, 0)
    pass_through(gpu)
