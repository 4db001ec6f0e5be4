"""What a user of this package has it do, as timed cases.

Each case is one pass through the public entry points at one size.  `listed`
holds the cases, `draw` makes more of the same kinds and ranges, `prepare`
makes what a program holds before the call, `run` is the pass, `work` the
bytes and operations that the pass cannot do without, `exact` the result in
64-bit arithmetic and `tolerance` how far a correct result may lie from it.

Kinds of case:
  step      one pruning step of a deployed backbone: select/pack with the
            attention plan, then one attention layer on the packed tokens
  chain     the step with the actor's decode before it, nothing read back by
            the host: gate, budget decode, select/pack + plan, attention
  cascade   several pruning steps in a row, each on the packed output of the
            one before
  layer     one attention layer of a layout whose plan is already there (every
            layer between two pruning steps)
  attn      the plain attention call on a packed buffer, plan and workspace
            made by the call
  residual  pruning after the attention residual: the kept rows of h + a
  select    select/pack with the plan, without the attention
  flops     FLOP accounting of an evaluation set's token trajectories
  pl        training: a Plackett-Luce draw and its log-probability, and the
            same draw scored under another policy
  readout   the LC1 readout of a classifier on the packed tokens
"""
import math

import numpy as np
import torch

import paper_2609_34325_amd as dora

D = 64  # head dimension of every backbone here
DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}


def listed():
    return [
        # The smallest call: DeiT-Tiny in fp32, four images (latency and launches).
        dict(name="step_tiny_f32", kind="step", B=4, N=197, H=3, dtype="f32", keep="uniform"),
        # DeiT-S serving batch from the actor's outputs on; four launches in a row.
        dict(name="chain_small_bf16", kind="chain", B=64, N=197, H=6, dtype="bf16"),
        # DeiT-B, the usual throughput batch.
        dict(name="step_base_bf16", kind="step", B=256, N=197, H=12, dtype="bf16", keep="beta"),
        # ViT-L with three pruning steps.
        dict(name="cascade_large_bf16", kind="cascade", B=256, N=197, H=16, dtype="bf16", keep="cascade", rounds=3),
        # ViT-B at 384 pixels, half of the images hardly pruned and half hard.
        dict(name="layer_384_bf16", kind="layer", B=64, N=577, H=12, dtype="bf16", keep="skew"),
        # High-resolution inputs: few, long and uneven sequences.
        dict(name="attn_highres_bf16", kind="attn", B=16, N=4096, H=12, dtype="bf16", keep="wide"),
        # DeiT-B layer in full precision (checking a deployment, or training in fp32).
        dict(name="layer_base_f32", kind="layer", B=64, N=197, H=12, dtype="f32", keep="beta"),
        # DeiT-B, rows deleted between the attention residual and the MLP.
        dict(name="residual_base_bf16", kind="residual", B=256, N=197, H=12, dtype="bf16", keep="beta"),
        # A whole evaluation shard at once: past the batch that one launch scans.
        dict(name="select_many_bf16", kind="select", B=8192, N=197, H=12, dtype="bf16", keep="beta"),
        # FLOPs of the ImageNet validation set's 50,000 trajectories, DeiT-B.
        dict(name="flops_eval", kind="flops", B=50000, N=197, L=12, C=768),
        # Policy update on ViT-B/384 rows.
        dict(name="pl_train_384", kind="pl", B=256, N=577),
        # DINOv2-B/14 readout.
        dict(name="readout_dinov2_bf16", kind="readout", B=256, N=257, H=12, dtype="bf16", keep="beta"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("step", "chain", "cascade", "layer", "attn", "residual", "select", "flops", "pl", "readout",
                       "step", "layer"))
    if kind == "flops":
        return dict(kind=kind, B=_log(rng, 64, 50000), N=rng.choice((50, 197, 257, 577)), L=rng.choice((6, 12, 24)),
                    C=rng.choice((192, 384, 768, 1024)))
    if kind == "pl":
        return dict(kind=kind, B=_log(rng, 1, 512), N=_log(rng, 17, 2048))
    H = rng.choice((3, 6, 12, 16))
    dtype = rng.choice(("bf16", "bf16", "bf16", "f32"))
    if kind == "attn":  # long sequences; at most 2^30 (2^26 in fp32) pairs of rows over all heads
        pairs = 1 << (30 if dtype == "bf16" else 26)
        N = min(_log(rng, 512, 16384), int(math.sqrt(pairs / H)))
        B = min(_log(rng, 1, 32), pairs // (N * N * H))
        return dict(kind=kind, B=B, N=N, H=H, dtype=dtype, keep=rng.choice(("wide", "beta")))
    if kind == "select":  # beyond 2048 images too; at most 1.6 M input rows
        N = _log(rng, 50, 1024)
        return dict(kind=kind, B=min(_log(rng, 512, 8192), 1600000 // N), N=N, H=H if N < 500 else 6,
                    dtype="bf16", keep=rng.choice(("uniform", "beta", "skew")))
    N = rng.choice((rng.randint(50, 200), rng.randint(197, 600), _log(rng, 17, 1024)))
    case = dict(kind=kind, B=min(_log(rng, 1, 400), 120000 // N), N=N, H=H, dtype=dtype,
                keep=rng.choice(("uniform", "beta", "skew")))
    if dtype == "f32" and kind in ("step", "chain", "cascade", "layer"):
        case["B"] = min(case["B"], 64, max(1, 24000 // N))
    if kind == "chain":
        del case["keep"]
        case["N"] = max(N, 17)
    if kind == "cascade":
        case["keep"], case["rounds"] = "cascade", rng.randint(2, 3)
    return case


# ------------------------------------------------------------------ inputs


def _keep_counts(rule, n, rng):
    """Keep counts (CLS included) of images of n tokens; at least four visual tokens stay."""
    B = len(n)
    if rule == "uniform":
        r = rng.uniform(0.1, 1.0, B)
    elif rule == "beta":
        r = 0.3 + 0.7 * rng.beta(4.0, 3.0, B)
    elif rule == "cascade":
        r = rng.uniform(0.6, 0.95, B)
    elif rule == "wide":
        r = rng.uniform(0.25, 1.0, B)
    else:  # skew: half hardly pruned, half hard
        high = rng.permutation(B) < (B + 1) // 2
        r = np.where(high, rng.uniform(0.90, 1.00, B), rng.uniform(0.08, 0.15, B))
    return np.clip(np.rint(r * n), np.minimum(n, 5), n).astype(np.int32)


def _with_total(counts, total, lo, hi, rng):
    """The counts with one more or one less here and there, so that they add up to `total`."""
    counts = counts.copy()
    while True:
        off = total - int(counts.sum())
        if off == 0:
            return counts
        room = np.flatnonzero(counts < hi if off > 0 else counts > lo)
        some = rng.permutation(room)[:abs(off)]
        counts[some] += 1 if off > 0 else -1


def _keeps(case, rng):
    """Keep counts of each round.  Every seed has other counts with the same total (the packed buffers' rows)."""
    rounds, fixed = [], np.random.default_rng(0)
    n = n_fixed = np.full(case["B"], case["N"], dtype=np.int32)
    for _ in range(case.get("rounds", 1)):
        n_fixed = _keep_counts(case["keep"], n_fixed, fixed)
        n = _with_total(_keep_counts(case["keep"], n, rng), int(n_fixed.sum()), np.minimum(n, 5), n, rng)
        rounds.append(n)
    return rounds


def _draw_counts(case, rng):
    """Plackett-Luce draws per image."""
    B, N = case["B"], case["N"]
    return np.minimum(2 * rng.integers(1, max(2, N // 3), B), N - 1).astype(np.int32)


def _cu(keep):
    return np.concatenate([[0], np.cumsum(keep, dtype=np.int64)]).astype(np.int32)


class _Source:
    """Random inputs on the GPU, from the seed alone."""

    def __init__(self, seed):
        self.np = np.random.default_rng(seed)
        self.gen = torch.Generator(device="cuda")
        self.gen.manual_seed(seed)

    def normal(self, shape, dtype=torch.float32, scale=1.0):
        x = torch.empty(shape, dtype=dtype, device="cuda")
        return x.normal_(0.0, scale, generator=self.gen)

    def uniform(self, shape, lo=0.0, hi=1.0):
        return torch.empty(shape, dtype=torch.float32, device="cuda").uniform_(lo, hi, generator=self.gen)

    def dev(self, a):
        return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _inputs(case, seed):
    """The inputs of one pass, without any of the package's own objects."""
    s, x, kind = _Source(seed), {}, case["kind"]
    B, N = case["B"], case["N"]
    if kind == "flops":
        t = np.empty((case["L"] + 1, B), dtype=np.int32)  # most blocks remove nothing, some remove a few tokens
        t[:2] = N
        for l in range(2, case["L"] + 1):
            cut = np.where(s.np.random(B) < 0.3, 2 * s.np.integers(1, 20, B), 0)
            t[l] = np.maximum(t[l - 1] - cut, np.minimum(t[l - 1], 5))
        x["tokens"] = s.dev(t)
        return x
    if kind == "pl":
        x["scores"], x["scores2"] = s.normal((B, N)), s.normal((B, N))
        u = s.uniform((B, N)).clamp_(1e-12, 1.0 - 1e-7)
        x["gumbel"] = -torch.log(-torch.log(u))
        total = int(_draw_counts(case, np.random.default_rng(0)).sum())
        k = _with_total(_draw_counts(case, s.np), total, 0, N - 1, s.np)
        x["k"], x["total"] = s.dev(k), int(k.sum())
        return x
    dt, C = DTYPES[case["dtype"]], case["H"] * D
    if kind == "chain":
        M = max(1, (N - 5) // 2)
        x["p_gate"], x["removal"] = s.uniform((B,)), s.normal((B, N))
        x["logits"], x["M"] = s.normal((B, M)), M
        x["tokens"] = s.normal((B, N, C), dt)
        x["qkv"] = [s.normal((B * N, case["H"], D), dt) for _ in range(3)]
        return x
    if kind == "cascade":
        n, rounds = np.full(B, N, dtype=np.int32), []
        x["tokens"] = s.normal((B, N, C), dt)
        for r, keep in enumerate(_keeps(case, s.np)):
            total = int(keep.sum())
            scores = s.normal((B, N) if r == 0 else (int(n.sum()),))
            rounds.append(dict(keep=s.dev(keep), total=total, max=int(keep.max()), scores=scores, n=n,
                               qkv=[s.normal((total, case["H"], D), dt) for _ in range(3)]))
            n = keep
        x["rounds"] = rounds
        return x
    keep = _keeps(case, s.np)[0]
    x["keep_np"], x["total"], x["max"] = keep, int(keep.sum()), int(keep.max())
    if kind in ("step", "residual", "select"):
        x["keep"], x["scores"] = s.dev(keep), s.normal((B, N))
        x["tokens"] = s.normal((B, N, C), dt)
    else:
        x["cu"] = s.dev(_cu(keep))
    if kind == "residual":
        x["a"] = s.normal((B, N, C), dt, 0.5)
    if kind in ("step", "layer", "attn"):
        x["qkv"] = [s.normal((x["total"], case["H"], D), dt) for _ in range(3)]
    if kind == "readout":  # rows with channel biases and scales, as residual streams have
        rows = s.normal((x["total"], C)) * s.uniform((C,), 0.5, 2.0) + s.normal((C,))
        x["x"], x["gamma"], x["beta"] = rows.to(dt), s.uniform((C,), 0.5, 1.5), s.normal((C,), scale=0.1)
    return x


# ------------------------------------------------------------------ passes


def _pack_outputs(case, total):
    dt = DTYPES[case["dtype"]]
    return dict(idx_out=torch.zeros(total, dtype=torch.int32, device="cuda"),
                cu_out=torch.zeros(case["B"] + 1, dtype=torch.int32, device="cuda"),
                packed_out=torch.zeros((total, case["H"] * D), dtype=dt, device="cuda"), cap_rows=total)


def prepare(case, seed):
    """A program's inputs, output buffers, workspaces and plans."""
    x, kind, B = _inputs(case, seed), case["kind"], case["B"]
    st = dict(case=case, x=x, status=dora.new_status())
    if kind in ("step", "chain", "select"):
        total = x["total"] if kind != "chain" else B * case["N"]
        st["pack"] = _pack_outputs(case, total)
        st["max"] = x["max"] if kind != "chain" else case["N"]
        st["total"] = total
        st["ws"] = dora.new_workspace(B, case["H"], st["max"])
        if kind != "select":
            st["out"] = torch.zeros_like(x["qkv"][0])
    elif kind == "residual":
        st["pack"] = _pack_outputs(case, x["total"])
    elif kind == "cascade":
        for r in x["rounds"]:
            r["pack"] = _pack_outputs(case, r["total"])
            r["ws"] = dora.new_workspace(B, case["H"], r["max"])
            r["out"] = torch.zeros_like(r["qkv"][0])
    elif kind == "layer":
        st["ws"] = dora.new_workspace(B, case["H"], x["max"])
        dora.dora_varlen_attn_plan(x["cu"], case["H"], x["max"], x["total"], st["ws"], st["status"])
        st["out"] = torch.zeros_like(x["qkv"][0])
    elif kind == "readout":
        st["ws"] = dora.new_lc1_workspace(B, case["H"] * D)
    if kind == "chain":
        st["rank"], st["list"] = (torch.zeros(B, dtype=torch.int32, device="cuda") for _ in range(2))
        st["n_on"] = torch.zeros(1, dtype=torch.int32, device="cuda")
        st["keep"], st["scores"] = torch.zeros(B, dtype=torch.int32, device="cuda"), torch.zeros_like(x["removal"])
    return st


def run(state):
    case, x, status = state["case"], state["x"], state["status"]
    kind = case["kind"]
    if kind == "flops":
        return dora.dora_trajectory_flops(x["tokens"], case["C"], case["N"] - 1, 16)
    if kind == "pl":
        order, cu, lp, status = dora.dora_pl_sample(x["scores"], x["gumbel"], x["k"], cap=x["total"])
        lp2, status = dora.dora_pl_logprob(x["scores2"], order, cu, dev_status=status)
        return order, cu, lp, lp2, status
    H = case["H"]
    if kind in ("step", "select"):
        idx, cu, packed, _ = dora.dora_select_pack_plan(x["scores"], x["keep"], x["tokens"], H, state["max"],
                                                        state["total"], state["ws"], dev_status=status, **state["pack"])
        if kind == "select":
            return idx, cu, packed, status
        out = dora.dora_varlen_attn_execute(*x["qkv"], cu, state["max"], state["ws"], out=state["out"],
                                            dev_status=status)
        return idx, cu, packed, out, status
    if kind == "chain":
        dora.dora_actor_gate(x["p_gate"], x["M"], case["N"], on_rank=state["rank"], on_list=state["list"],
                             n_on=state["n_on"], dev_status=status)
        keep, scores, _ = dora.dora_actor_decode(x["logits"], state["rank"], case["N"], x["removal"],
                                                 keep_out=state["keep"], scores_out=state["scores"], dev_status=status)
        idx, cu, packed, _ = dora.dora_select_pack_plan(scores, keep, x["tokens"], H, state["max"], state["total"],
                                                        state["ws"], dev_status=status, **state["pack"])
        out = dora.dora_varlen_attn_execute(*x["qkv"], cu, state["max"], state["ws"], out=state["out"],
                                            dev_status=status)
        return state["rank"], state["list"], state["n_on"], keep, scores, idx, cu, packed, out, status
    if kind == "cascade":
        tokens, cu_in, outs = x["tokens"], None, []
        for r in x["rounds"]:
            idx, cu, packed, _ = dora.dora_select_pack_plan(r["scores"], r["keep"], tokens, H, r["max"], r["total"],
                                                            r["ws"], cu_in=cu_in, N=case["N"], dev_status=status,
                                                            **r["pack"])
            out = dora.dora_varlen_attn_execute(*r["qkv"], cu, r["max"], r["ws"], out=r["out"], dev_status=status)
            outs.append((idx, cu, packed, out))
            tokens, cu_in = packed, cu
        return outs, status
    if kind == "layer":
        return dora.dora_varlen_attn_execute(*x["qkv"], x["cu"], x["max"], state["ws"], out=state["out"],
                                             dev_status=status), status
    if kind == "attn":
        return dora.dora_varlen_attn(*x["qkv"], x["cu"], x["max"])
    if kind == "residual":
        return dora.dora_select_pack_residual(x["scores"], x["keep"], x["tokens"], x["a"], dev_status=status,
                                              **state["pack"])
    return dora.dora_lc1_readout(x["x"], x["cu"], x["gamma"], x["beta"], 1e-6, workspace=state["ws"])


# ------------------------------------------------------------------ work


def _attn_work(lens, H, elt):
    lens = np.asarray(lens, dtype=np.float64)
    return 4.0 * lens.sum() * H * D * elt, 4.0 * D * H * float((lens ** 2).sum())


def _select_bytes(total, B, n_in, C, elt):
    return 2.0 * total * C * elt + 4.0 * (n_in + total + 2 * B + 1)


def work(case):
    kind, B, N = case["kind"], case["B"], case["N"]
    if kind == "flops":
        return dict(bytes=4.0 * (case["L"] + 1) * B + 8.0 * B + 8, flops=30.0 * case["L"] * B)
    if kind == "pl":
        drawn = float(_draw_counts(case, np.random.default_rng(0)).sum())
        return dict(bytes=12.0 * B * N + 8.0 * drawn + 20.0 * B, flops=B * N * (math.log2(max(N, 2)) + 20.0))
    H, elt = case["H"], 2 if case["dtype"] == "bf16" else 4
    C = H * D
    if kind == "chain":
        M = max(1, (N - 5) // 2)
        # gates open for half of the images; an open one keeps about half of its tokens
        keep = np.where(np.arange(B) % 2 == 0, N, np.linspace(5, N - 2, B))
        ab, af = _attn_work(keep, H, elt)
        return dict(bytes=4.0 * (4 * B + B * M / 2 + 2 * B * N) + _select_bytes(keep.sum(), B, B * N, C, elt) + ab,
                    flops=af)
    if kind == "cascade":
        n, nbytes, flops = np.full(B, N, dtype=np.int32), 0.0, 0.0
        for keep in _keeps(case, np.random.default_rng(0)):
            ab, af = _attn_work(keep, H, elt)
            nbytes += _select_bytes(float(keep.sum()), B, float(n.sum()), C, elt) + ab
            flops += af
            n = keep
        return dict(bytes=nbytes, flops=flops)
    keep = _keeps(case, np.random.default_rng(0))[0]  # they vary with the seed, their total does not
    total = float(keep.sum())
    if kind in ("layer", "attn"):
        ab, af = _attn_work(keep, H, elt)
        return dict(bytes=ab, flops=af)
    if kind == "residual":
        return dict(bytes=_select_bytes(total, B, B * N, C, elt) + total * C * elt, flops=total * C)
    if kind == "readout":
        return dict(bytes=total * C * elt + 8.0 * B * C + 8.0 * C + 4.0 * (B + 1), flops=8.0 * total * C)
    sb = _select_bytes(total, B, B * N, C, elt)
    if kind == "select":
        return dict(bytes=sb, flops=0.0)
    ab, af = _attn_work(keep, H, elt)
    return dict(bytes=sb + ab, flops=af)


# ------------------------------------------------------------------ results


def tolerance(case):
    """About four times the largest distance from `exact` seen over the listed and fifteen drawn cases."""
    kind = case["kind"]
    if kind in ("flops", "select", "residual"):  # whole numbers, copied bytes, one rounding of an exact sum
        return "exact"
    if kind == "pl":  # seen: rel 6e-8, max 1.5e-7; up to 2047 fp32 logarithms are added
        return {"rel": 5e-7, "max": 2e-6}
    if kind == "readout":  # seen: rel 7e-8, max 3e-7
        return {"rel": 3e-7, "max": 1.5e-6}
    if case["dtype"] == "f32":  # seen: rel 3.4e-7, max 6e-6
        return {"rel": 1.5e-6, "max": 2.5e-5}
    # seen: rel 2.3e-3, max 2e-2 (probabilities rounded to bf16 for the second product, the output to bf16)
    return {"rel": 1e-2, "max": 8e-2}


def _exact_attn(qkv, lens):
    q, k, v = qkv
    out = torch.zeros(q.shape, dtype=torch.float64, device=q.device)
    r = 0
    for n in (int(n) for n in lens):
        for h0 in range(0, q.shape[1], max(1, (1 << 28) // (n * n + 1))):
            h1 = min(q.shape[1], h0 + max(1, (1 << 28) // (n * n + 1)))
            qs, ks, vs = (t[r:r + n, h0:h1].double().transpose(0, 1).contiguous() for t in (q, k, v))
            p = torch.softmax(torch.bmm(qs, ks.transpose(1, 2).contiguous()) / math.sqrt(D), dim=2)
            out[r:r + n, h0:h1] = torch.bmm(p, vs).transpose(0, 1)
        r += n
    return out


def _exact_select(scores, keep, rows, lens):
    """Indices of CLS and the keep - 1 highest scores of each image in ascending order, and the rows they name.
    scores, rows: all images' tokens one after the other, lens of them each."""
    idx, src, r = [], [], 0
    for k, n in zip(keep, lens):
        k, n = int(k), int(n)
        by_score = torch.sort(scores[r + 1:r + n], descending=True, stable=True).indices[:k - 1] + 1
        kept = torch.cat([torch.zeros(1, dtype=torch.int64, device=scores.device), torch.sort(by_score).values])
        idx.append(kept)
        src.append(kept + r)
        r += n
    idx = torch.cat(idx)
    return idx.to(torch.int32), rows[torch.cat(src)]


def _padded(t, rows):
    out = torch.zeros((rows,) + tuple(t.shape[1:]), dtype=t.dtype, device=t.device)
    out[:t.shape[0]] = t
    return out


def _exact_logprob(scores, order, k):
    """Ordered log-probability of each image's draws: order holds them one image after the other."""
    out, r = [], 0
    for b, n in enumerate(int(v) for v in k):
        s = scores[b, 1:].double()
        drawn = order[r:r + n].long() - 1
        left = torch.ones(s.numel(), dtype=torch.bool, device=s.device)
        left[drawn] = False
        terms = torch.cat([s[left], s[drawn].flip(0)])  # the last draw after all that stay, the first draw last
        denom = torch.logcumsumexp(terms, 0).flip(0)[:n]
        out.append((s[drawn] - denom).sum())
        r += n
    return torch.stack(out)


def exact(case, seed):
    x, kind, B, N = _inputs(case, seed), case["kind"], case["B"], case["N"]
    status = torch.zeros(1, dtype=torch.int32, device="cuda")
    if kind in ("flops", "select"):
        return None  # whole numbers and copied bytes
    if kind == "pl":
        keys = (x["scores"] + x["gumbel"])[:, 1:]  # compared in 32 bits, equal keys by the higher position
        rev = torch.sort(keys.flip(1), dim=1, descending=True, stable=True).indices
        draws = (N - 1) - rev
        k = x["k"].cpu().numpy()
        order = torch.cat([draws[b, :int(k[b])] for b in range(B)])
        cu = torch.from_numpy(_cu(k)).cuda()
        return (order.to(torch.int32), cu, _exact_logprob(x["scores"], order, k),
                _exact_logprob(x["scores2"], order, k), status)
    dense = [N] * B
    if kind == "chain":
        legal = min(max((N - 5) // 2, 0), x["M"])
        on = (x["p_gate"] >= 0.5) & (legal > 0)
        rank = torch.where(on, torch.cumsum(on, 0) - 1, torch.full_like(on, -1, dtype=torch.int64))
        on_list = torch.full((B,), -1, dtype=torch.int32, device="cuda")
        on_list[:int(on.sum())] = torch.nonzero(on).flatten().to(torch.int32)
        best = torch.argmax(x["logits"][:, :max(legal, 1)], dim=1)
        keep = torch.where(on, N - 2 * (best[rank.clamp(min=0)] + 1), torch.full_like(rank, N))
        lens = keep.cpu().numpy()
        cu = torch.from_numpy(_cu(lens)).cuda()
        idx, packed = _exact_select(-x["removal"].flatten(), lens, x["tokens"].flatten(0, 1), dense)
        out = _padded(_exact_attn([t[:int(lens.sum())] for t in x["qkv"]], lens), B * N)
        return (rank.to(torch.int32), on_list, on.sum().to(torch.int32).reshape(1), keep.to(torch.int32),
                -x["removal"], _padded(idx, B * N), cu, _padded(packed, B * N), out, status)
    if kind == "cascade":
        rows, outs = x["tokens"].flatten(0, 1), []
        for r in x["rounds"]:
            lens = r["keep"].cpu().numpy()
            idx, rows = _exact_select(r["scores"].flatten(), lens, rows, r["n"])
            outs.append((idx, torch.from_numpy(_cu(lens)).cuda(), rows, _exact_attn(r["qkv"], lens)))
        return outs, status
    lens = x["keep_np"]
    if kind in ("layer", "attn"):
        out = _exact_attn(x["qkv"], lens)
        return out if kind == "attn" else (out, status)
    cu = torch.from_numpy(_cu(lens)).cuda()
    if kind == "readout":
        rows = x["x"].double()
        mu = rows.mean(1, keepdim=True)
        var = ((rows - mu) ** 2).mean(1, keepdim=True)
        y = (rows - mu) / torch.sqrt(var + 1e-6) * x["gamma"].double() + x["beta"].double()
        at, halves = _cu(lens), []
        for b in range(B):
            halves.append(torch.cat([y[at[b]], y[at[b] + 1:at[b + 1]].mean(0)]))
        return torch.stack(halves), status
    if kind == "residual":
        rows = (x["tokens"].double() + x["a"].double()).flatten(0, 1)
        idx, packed = _exact_select(x["scores"].flatten(), lens, rows, dense)
        return idx, cu, packed, status
    idx, packed = _exact_select(x["scores"].flatten(), lens, x["tokens"].flatten(0, 1), dense)
    return idx, cu, packed, _exact_attn(x["qkv"], lens), status
