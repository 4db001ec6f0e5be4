"""fp32 attention from split bf16 products (GPU): tile, stage and part edges on
both launch forms, and values that the split cannot represent."""
import numpy as np
import pytest
import torch

import oracle
import workloads
from gpu_util import cu_of, to_dev

pytestmark = pytest.mark.gpu

# One rounding of fp32 sums is 6e-8 of the result; scores carry an absolute
# error of about 64 roundings of |q||k| / 64 <= 64 * 6e-8 * 2, so each weight
# is within 8e-6 of its value relatively, and the output of its rms.
REL = 1e-5
LENS = [1, 15, 16, 17, 31, 32, 33, 63, 64, 65, 95, 96, 97, 128, 129, 160, 161, 191, 192, 193, 224, 225, 400]


def run(gpu, q, k, v, lens):
    cu = cu_of(lens)
    out = gpu.dora_varlen_attn(to_dev(q), to_dev(k), to_dev(v), to_dev(cu), int(max(lens)))
    torch.cuda.synchronize()
    return out.cpu().numpy().astype(np.float64), cu


def close(got, want, what=""):
    rms = np.sqrt((want ** 2).mean())
    assert np.all(np.isfinite(got)), what
    assert np.abs(got - want).max() <= REL * max(rms, np.abs(want).max() / 16), (what, np.abs(got - want).max(), rms)


# heads * sequences * 3 chunks: 23 * 12 items and more, or 1 * 3 a call (split while 3 items per workgroup fit)
@pytest.mark.parametrize("H", [1, 12])
def test_edges(gpu, H):
    rng = np.random.default_rng(H)
    groups = [LENS] if H > 1 else [LENS[i:i + 4] for i in range(0, len(LENS), 4)]
    for lens in groups:
        q, k, v = workloads.random_qkv(rng, lens, H, "f32")
        got, cu = run(gpu, q, k, v, lens)
        close(got, oracle.varlen_attn(q, k, v, cu, "f32"), lens)


@pytest.mark.parametrize("n", [40, 210])
@pytest.mark.parametrize("B", [1, 64])
def test_values_past_the_split(gpu, n, B):
    """Infinities, NaN and the largest values give what fp32 arithmetic gives;
    V near the smallest normal numbers keeps its relative precision."""
    H, lens = 2, [n] * B
    rng = np.random.default_rng(n + B)
    q0, k0, v0 = workloads.random_qkv(rng, lens, H, "f32")
    b, j = B - 1, n - 3                       # the row of the last sequence that is changed
    row = b * n + j

    # a key of score -inf has weight 0: the sequence without it
    q, k = q0.copy(), k0.copy()
    q[:, 0, 0] = 1.0
    k[row, 0, 0] = -np.inf
    got, _ = run(gpu, q, k, v0, lens)
    keep = np.delete(np.arange(b * n, b * n + n), j)
    sub, cu = [np.ascontiguousarray(t[keep]) for t in (k, v0)], cu_of([n - 1])
    want = oracle.varlen_attn(np.ascontiguousarray(q[keep]), *sub, cu, "f32")
    close(got[keep][:, 0], want[:, 0])

    # one infinite, one NaN and one huge value in V reach their own dimensions only
    v, vz = v0.copy(), v0.copy()
    for d, x in ((3, np.inf), (5, np.nan), (9, np.finfo(np.float32).max)):
        v[row, 1, d], vz[row, 1, d] = x, 0.0
    got, cu = run(gpu, q0, k0, v, lens)
    want = oracle.varlen_attn(q0, k0, vz, cu, "f32")
    seq = slice(b * n, b * n + n)
    assert np.all(got[seq, 1, 3] == np.inf) and np.all(np.isnan(got[seq, 1, 5]))
    one = np.zeros_like(v0)
    one[row, 1, 9] = 1.0
    weight = oracle.varlen_attn(q0, k0, one, cu, "f32")[seq, 1, 9] * np.float64(np.finfo(np.float32).max)
    assert np.abs(got[seq, 1, 9] / weight - 1).max() <= REL
    got[seq, 1, [[3], [5], [9]]] = want[seq, 1, [[3], [5], [9]]] = 0.0
    close(got, want)

    # a NaN query spoils its own row only
    q = q0.copy()
    q[row, 0, 7] = np.nan
    got, cu = run(gpu, q, k0, v0, lens)
    want = oracle.varlen_attn(q0, k0, v0, cu, "f32")
    assert np.all(np.isnan(got[row, 0]))
    got[row, 0] = want[row, 0] = 0.0
    close(got, want)

    # tiny and large V
    for scale in (2.0 ** -115, 2.0 ** 90, 2.0 ** 120):
        v = v0 * np.float32(scale)
        got, cu = run(gpu, q0, k0, v, lens)
        close(got / scale, oracle.varlen_attn(q0, k0, v0, cu, "f32"), scale)


@pytest.mark.parametrize("B", [1, 64])                      # split and whole items
@pytest.mark.parametrize("how", ["infinite", "overflow"])   # an infinite key, or finite factors whose product is
@pytest.mark.parametrize("lead", [1, 15, 16, 17, 31, 32, 33, 63, 64, 96, 130, 209])
def test_leading_keys_of_score_minus_infinity(gpu, lead, how, B):
    """The first `lead` keys of a sequence score -inf: weight 0, the sequence without
    them.  A sequence whose every score is -inf is NaN, as softmax gives."""
    H, n = 2, 210
    lens = [n] * B
    rng = np.random.default_rng(lead)
    q, k, v = workloads.random_qkv(rng, lens, H, "f32")
    row0 = (B - 1) * n
    k[row0:row0 + n, 0, 0] = 0.0
    q[row0:row0 + n, 0, 0], k[row0:row0 + lead, 0, 0] = (1.0, -np.inf) if how == "infinite" else (2.0 ** 100, -2.0 ** 100)
    got, _ = run(gpu, q, k, v, lens)
    qs = q[row0:row0 + n].copy()
    qs[:, 0, 0] = 0.0                          # times zero for the keys that stay
    want = oracle.varlen_attn(np.ascontiguousarray(qs[lead:]), np.ascontiguousarray(k[row0 + lead:row0 + n]),
                              np.ascontiguousarray(v[row0 + lead:row0 + n]), cu_of([n - lead]), "f32")
    close(got[row0 + lead:row0 + n, 0], want[:, 0], (lead, how))
    k[row0:row0 + n, 0, 0] = k[row0, 0, 0]
    got, _ = run(gpu, q, k, v, lens)
    assert np.all(np.isnan(got[row0:row0 + n, 0])) and np.all(np.isfinite(got[row0:row0 + n, 1]))


@pytest.mark.parametrize("B", [1, 64])                # split and whole items
@pytest.mark.parametrize("e", [100, 109, 110, 111, 114, 118, 120])
@pytest.mark.parametrize("small", ["q", "k"])
def test_small_factors_of_large_ones(gpu, small, e, B):
    """Q near 2^-e against K near 2^e and the other way round: ordinary scores, of
    which no bit of the small factor may be missing.  One sequence of the batch."""
    H, n = 2, 210
    lens = [n] * B
    q, k, v = workloads.random_qkv(np.random.default_rng(e), lens, H, "f32")
    s = slice((B - 1) * n, B * n)
    for t in (q, k):                                  # at least 2^-5: normal numbers after the scaling
        t[s] = np.copysign(np.maximum(np.abs(t[s]), 2.0 ** -5), t[s])
    q[s] *= np.float32(2.0 ** (-e if small == "q" else e))
    k[s] *= np.float32(2.0 ** (e if small == "q" else -e))
    got, cu = run(gpu, q, k, v, lens)
    close(got, oracle.varlen_attn(q, k, v, cu, "f32"), (small, e))


@pytest.mark.parametrize("B", [1, 64])
@pytest.mark.parametrize("x", [100, 110, 118, 122, 125])
def test_small_weights_of_large_values(gpu, x, B):
    """One key of weight 1 and value 0, all others of weight near 2^-x and positive
    values: what the small weights say is the whole result."""
    H, n = 2, 210
    lens = [n] * B
    q, k, v = workloads.random_qkv(np.random.default_rng(x), lens, H, "f32")
    q[:, :, 0], k[:, :, 0] = 8.0, -np.float32(x * np.log(2.0))
    q[:, :, 1:] *= np.float32(0.05)
    k[n // 2::n, :, 0], k[n // 2::n, :, 1:] = 0.0, 0.0
    v = (np.abs(v) + np.float32(0.1)) * np.float32(2.0 ** 80)
    v[n // 2::n] = 0.0
    got, cu = run(gpu, q, k, v, lens)
    want = oracle.varlen_attn(q, k, v, cu, "f32")
    # exp2's argument is up to 126 and carries about 6 roundings of 6e-8: 126 ln 2 * 6 * 6e-8 = 3.1e-5 of a weight
    assert np.abs(got / want - 1).max() <= 4e-5


@pytest.mark.parametrize("H", [1, 12])
def test_recomputed_tiles_edges(gpu, H):
    """Every tile through the fp32 matrix instructions (V past the split's range)."""
    rng = np.random.default_rng(H + 40)
    groups = [LENS] if H > 1 else [LENS[i:i + 4] for i in range(0, len(LENS), 4)]
    for lens in groups:
        q, k, v = workloads.random_qkv(rng, lens, H, "f32")
        got, cu = run(gpu, q, k, v * np.float32(2.0 ** 115), lens)
        close(got / 2.0 ** 115, oracle.varlen_attn(q, k, v, cu, "f32"), lens)


# (sequences, heads): split items, and 3 or more whole items per workgroup (tickets from the counters)
@pytest.mark.parametrize("B,H", [(2, 3), (64, 16)])
def test_one_plan_many_executes(gpu, B, H):
    """One plan for several layers, fp32 and bf16 in turn on one workspace: every
    layer writes every row, and the queue's counters are zero after each."""
    rng = np.random.default_rng(B)
    lens = rng.integers(1, 400, size=B)
    mx, total = int(lens.max()), int(lens.sum())
    q, k, v = workloads.random_qkv(rng, lens, H, "f32")
    cu = cu_of(lens)
    want = oracle.varlen_attn(q, k, v, cu, "f32")
    f32 = [to_dev(t) for t in (q, k, v)]
    bf16 = [t.bfloat16() for t in f32]
    ws, st, cu_d = gpu.new_workspace(B, H, mx), gpu.new_status(), to_dev(cu)
    gpu.dora_varlen_attn_plan(cu_d, H, mx, total, ws, st)
    first = {}
    for layer in range(6):
        x = bf16 if layer in (2, 3) else f32
        out = torch.full_like(x[0], -777.0)
        gpu.dora_varlen_attn_execute(*x, cu_d, mx, ws, out=out, dev_status=st)
        torch.cuda.synchronize()
        head = ws[:2048].view(torch.int32).cpu().numpy()
        assert int(st.item()) == 0 and np.all(head[64:64 + 32 * 9:32] == 0)   # eight ticket counters, the exit counter
        if x is f32:
            close(out.cpu().numpy().astype(np.float64), want, layer)
        else:  # inputs rounded to bf16: scores of up to 5 off by 2^-8, weights by 2 %, of values up to 4
            assert np.abs(out.float().cpu().numpy() - want).max() <= 0.1
        assert torch.equal(out, first.setdefault(x is f32, out))
