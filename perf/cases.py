"""Workloads of the tree-verify library for timing: what a serving loop asks of it, through the public entry points.

Kinds of a case
    step        one request's verify step: tree build, attention of every layer, greedy acceptance, KV commit
    attn        the attention of a target's layers alone (bf16 or FP8 cache)
    batch       a verify step of several requests of different lengths over a paged cache
    stochastic  the rejection walk at temperature 1
    lm_head     greedy acceptance straight from the final hidden states
    build       the draft tree alone, at a fixed or at an online budget

Every layer has a K/V cache of its own, as in a real target, so that caches are not met again within a pass; a few
layers stand for all of them.  Inputs are drawn on the GPU from the seed alone.
"""
import math
import random

import torch

from paper_2605_29727_amd import binding as btv
from paper_2605_29727_amd import synth

I32, F32, BF16, U8 = torch.int32, torch.float32, torch.bfloat16, torch.uint8
FP8_SCALE = 4.5 / 448.0          # the codes cover |x| <= 4.5 of N(0,1) values
VOCAB = 128256


def _case(kind, name=None, **sizes):
    c = {"kind": kind, **sizes}
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # The smallest step: one head, a 64-token vocabulary, fp32 throughout, launched call by call.  All latency.
        _case("step", "step_fp32_tiny", dtype="fp32", layers=1, L=128, N=16, Hq=1, Hkv=1, D=64, B=4, V=64, marg="sigma2",
              graph=False),
        # The step of an 8B-shaped target at an 8k context, recorded in a HIP graph as a serving loop does it.
        _case("step", "step_8b_L8192_N64", dtype="bf16", layers=4, L=8192, N=64, Hq=32, Hkv=8, D=128, B=16, V=VOCAB,
              marg="sigma5", graph=True),
        # One small layer with 64-channel heads, ragged in the context and in the tree, one eager call.
        _case("attn", "attn_d64_L1531_N23", kv="bf16", layers=1, L=1531, N=23, Hq=32, Hkv=8, D=64, tree="random"),
        # The largest tree on the 8B shape.
        _case("attn", "attn_8b_L8192_N256", kv="bf16", layers=4, L=8192, N=256, Hq=32, Hkv=8, D=128, tree="random"),
        # The largest call: a 70B-shaped target at a 32k context.
        _case("attn", "attn_70b_L32768_N128", kv="bf16", layers=16, L=32768, N=128, Hq=64, Hkv=8, D=128, tree="deep"),
        # FP8 cache, odd context length and tree size.
        _case("attn", "attn_fp8_8b_L12003_N33", kv="fp8", layers=4, L=12003, N=33, Hq=32, Hkv=8, D=128, tree="random"),
        # A ragged batch over a paged cache: 8 requests of 1k to 16k context with trees of 32 to 128 nodes.
        _case("batch", "batch8_paged", kv="bf16", layers=2, requests=8, L_lo=1024, L_hi=16384, N_lo=32, N_hi=128, Hq=32, Hkv=8,
              D=128, B=16, V=VOCAB, mix=5),
        # Many short conversations with small trees, FP8 paged cache.
        _case("batch", "batch32_paged_fp8", kv="fp8", layers=2, requests=32, L_lo=100, L_hi=4000, N_lo=4, N_hi=24, Hq=32, Hkv=8,
              D=128, B=8, V=32000, mix=7),
        # A drafter that knows nothing: 127 children of the root, all of them tried.
        _case("stochastic", "stochastic_reject_N128", dtype="fp32", N=128, B=16, V=VOCAB, marg="sigma3", noise=-3.0),
        # A drafter that the target mostly agrees with: several levels are accepted.
        _case("stochastic", "stochastic_agree_N64", dtype="bf16", N=64, B=16, V=VOCAB, marg="drafter", noise=0.5),
        # LM head of the 8B shape fused with the argmax.
        _case("lm_head", "lm_head_8b_N64", N=64, h=4096, V=VOCAB),
        # The largest draft tree over a confident drafter's marginals: a deep one.
        _case("build", "build_deep_N256", N=256, B=16, V=VOCAB, marg="drafter", adaptive=False),
    ]


# ----------------------------------------------------------------------------------------------------------------------
# drawn cases
# ----------------------------------------------------------------------------------------------------------------------

HEADS = [(32, 8, 128), (64, 8, 128), (32, 8, 64), (16, 4, 64), (8, 2, 128), (8, 8, 64), (16, 2, 128)]
MOST_FLOPS = 4 * 64 * 128 * 128 * 32768 * 16        # of the largest listed case
MOST_BYTES = 2 * 32896 * 8 * 128 * 2 * 16


def _log(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _layers(rng, L, N, Hq, Hkv, D):
    """As many of 1, 2, 4, 8 layers as keep a pass below a quarter of the largest listed case."""
    fits = [n for n in (1, 2, 4, 8) if 4 * n * 4 * Hq * D * N * (L + N) <= MOST_FLOPS and 4 * n * 4 * (L + N) * Hkv * D <= MOST_BYTES]
    return rng.choice(fits or [1])


def draw(rng):
    kind = rng.choice(["step", "attn", "attn", "batch", "stochastic", "lm_head", "build"])
    marg = rng.choice(["sigma1", "sigma3", "sigma5", "drafter"])
    V = _log(rng, 1000, VOCAB)
    if kind == "step" and rng.random() < 0.25:
        Hkv = rng.choice([1, 2])
        return _case("step", dtype="fp32", layers=1, L=_log(rng, 16, 512), N=_log(rng, 2, 32), Hq=Hkv * rng.choice([1, 2, 4]), Hkv=Hkv,
                     D=rng.choice([64, 128]), B=rng.randint(2, 8), V=_log(rng, 64, 5000), marg="sigma2", graph=rng.random() < 0.5)
    Hq, Hkv, D = rng.choice(HEADS)
    if kind in ("step", "attn"):
        L, N = _log(rng, 64, 32768), _log(rng, 4, 256)
        layers = _layers(rng, L, N, Hq, Hkv, D)
        if kind == "step":
            return _case("step", dtype="bf16", layers=min(layers, 4), L=L, N=N, Hq=Hq, Hkv=Hkv, D=D, B=rng.randint(4, 16), V=V,
                         marg=marg, graph=rng.random() < 0.5)
        kv = "fp8" if D == 128 and rng.random() < 0.4 else "bf16"
        return _case("attn", kv=kv, layers=layers, L=L, N=N, Hq=Hq, Hkv=Hkv, D=D, tree=rng.choice(["random", "deep", "star", "binary"]))
    if kind == "batch":
        requests = _log(rng, 2, 32)
        kv = "fp8" if D == 128 and rng.random() < 0.4 else "bf16"
        Hq, Hkv = (32, 8) if D == 128 else (16, 4)
        L_hi, N_hi = _log(rng, 256, 120000 // requests if requests > 8 else 16384), _log(rng, 8, min(128, 1600 // requests))
        return _case("batch", kv=kv, layers=rng.choice([1, 2]), requests=requests, L_lo=max(1, L_hi // 16), L_hi=L_hi, N_lo=max(2, N_hi // 4),
                     N_hi=N_hi, Hq=Hq, Hkv=Hkv, D=D, B=rng.randint(4, 16), V=V, mix=rng.randint(1, 1 << 20))
    if kind == "stochastic":
        return _case("stochastic", dtype=rng.choice(["fp32", "bf16"]), N=_log(rng, 4, 200), B=rng.randint(4, 16), V=V, marg=marg,
                     noise=rng.choice([-3.0, -1.0, 0.25, 0.5, 1.0]))
    if kind == "lm_head":
        return _case("lm_head", N=_log(rng, 1, 256), h=128 * rng.randint(8, 32), V=_log(rng, 8000, VOCAB))
    return _case("build", N=_log(rng, 4, 256), B=rng.randint(2, 16), V=V, marg=marg, adaptive=rng.random() < 0.4)


# ----------------------------------------------------------------------------------------------------------------------
# inputs
# ----------------------------------------------------------------------------------------------------------------------

def _zeros(n, dtype=I32):
    return torch.zeros(n, dtype=dtype, device="cuda")


def _randn(g, shape, dtype):
    """N(0,1) rounded to `dtype`, drawn a slice of the first dimension at a time."""
    out = torch.empty(shape, dtype=dtype, device="cuda")
    for x in (out if len(shape) > 3 else (out,)):
        x.copy_(torch.randn(x.shape, generator=g, dtype=F32, device="cuda"))
    return out


def _kv(g, shape, kv):
    if kv != "fp8":
        return _randn(g, shape, F32 if kv == "fp32" else BF16)
    out = torch.empty(shape, dtype=U8, device="cuda")
    for x in out:
        y = torch.randn(x.shape, generator=g, dtype=F32, device="cuda").clamp_(-4.5, 4.5).div_(FP8_SCALE)
        x.copy_(y.to(torch.float8_e4m3fn).view(U8))
    return out


def _marginals(g, shape, marg):
    """Draft marginals [.., B, V]: softmax of normal logits, or those of a confident drafter (one token of probability
    0.9 * 0.93^k at position k, the rest softmax(3 N(0,1)))."""
    sigma = 3.0 if marg == "drafter" else float(marg[5:])
    m = torch.softmax(torch.randn(shape, generator=g, dtype=F32, device="cuda") * sigma, dim=-1)
    if marg == "drafter":
        B, V = shape[-2:]
        top = (0.9 * 0.93 ** torch.arange(B, device="cuda", dtype=F32)).expand(shape[:-1]).unsqueeze(-1)
        hot = torch.randint(0, V, tuple(shape[:-1]) + (1,), generator=g, device="cuda")
        m = m * (1.0 - top) / (1.0 - m.gather(-1, hot))
        m = m.scatter(-1, hot, top)
    return m.contiguous()


def _tree_out(N):
    return {"parent": _zeros(N), "token": _zeros(N), "depth": _zeros(N), "rho": _zeros(N, F32), "n_out": _zeros(1), "ahat": _zeros(1, F32)}


def _tree(marg, N):
    """A built tree, for inputs that follow from one."""
    B, V = marg.shape
    t = _tree_out(N)
    btv.btv_tree_build(marg, N, t["parent"], t["token"], t["depth"], t["rho"], t["n_out"], t["ahat"],
                       btv.alloc_workspace(btv.btv_tree_build_workspace(B, V, N)))
    return t


def _target_logits(g, best, V, dtype):
    """Greedy targets: N(0,1) logits in which 7 rows of 10 prefer token best[row], the drafter's own favourite there."""
    rows = best.numel()
    out = torch.empty((rows, V), dtype=dtype, device="cuda")
    for r0 in range(0, rows, 256):
        x = torch.randn((min(256, rows - r0), V), generator=g, dtype=F32, device="cuda")
        b = best[r0:r0 + 256].to(torch.int64).unsqueeze(1)
        x.scatter_add_(1, b, 8.0 * (torch.rand(b.shape, generator=g, device="cuda") < 0.7).to(F32))
        out[r0:r0 + 256] = x
    return out


def _lengths(case):
    """Context lengths and tree sizes of a batch's requests: part of the case, not of the seed."""
    r = random.Random(case["mix"])
    n = case["requests"]
    return ([r.randint(case["L_lo"], case["L_hi"]) for _ in range(n)], [r.randint(case["N_lo"], case["N_hi"]) for _ in range(n)])


# ----------------------------------------------------------------------------------------------------------------------
# one kind after the other: a function that makes the state and one that makes the pass
# ----------------------------------------------------------------------------------------------------------------------

def _prepare_step(c, g):
    dt = F32 if c["dtype"] == "fp32" else BF16
    layers, L, N, Hq, Hkv, D, B, V = (c[k] for k in ("layers", "L", "N", "Hq", "Hkv", "D", "B", "V"))
    marg = _marginals(g, (B, V), c["marg"])
    depth = torch.cat([_zeros(1), _tree(marg, N)["depth"]]).clamp(max=B - 1)
    s = {"c": c, "marg": marg, "logits": _target_logits(g, marg.argmax(1)[depth.long()], V, dt),
         "Q": _randn(g, (layers, N, Hq, D), dt), "K": _kv(g, (layers, L + N, Hkv, D), c["dtype"]), "V": _kv(g, (layers, L + N, Hkv, D), c["dtype"]),
         "path": _zeros(N), "n_acc": _zeros(1), "bonus": _zeros(1), "new_len": _zeros(1), "tree": _tree_out(N),
         "ws_build": btv.alloc_workspace(btv.btv_tree_build_workspace(B, V, N)),
         "ws_attn": btv.alloc_workspace(btv.btv_tree_verify_attn_workspace(N, L, Hq, Hkv, D, btv.BTV_F32 if dt == F32 else btv.BTV_BF16)),
         "ws_acc": btv.alloc_workspace(btv.btv_tree_accept_workspace(N, V, False))}
    s["O"] = torch.zeros_like(s["Q"])
    s["per_layer"] = [(s["Q"][i], s["K"][i], s["V"][i], s["O"][i]) for i in range(layers)]
    s["out"] = {**s["tree"], **{k: s[k] for k in ("O", "path", "n_acc", "bonus", "new_len", "K", "V")},
                "K_tree": s["K"][:, L:], "V_tree": s["V"][:, L:]}
    if c["graph"]:
        side, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            _run_step(s)
            with torch.cuda.graph(graph, stream=side):
                _run_step(s)
        torch.cuda.current_stream().wait_stream(side)
        s["graph"] = graph
    return s


def _run_step(s):
    c, t = s["c"], s["tree"]
    btv.btv_tree_build(s["marg"], c["N"], t["parent"], t["token"], t["depth"], t["rho"], t["n_out"], t["ahat"], s["ws_build"])
    for Q, K, V, O in s["per_layer"]:
        btv.btv_tree_verify_attn(Q, K, V, t["parent"], c["L"], O, s["ws_attn"])
    btv.btv_tree_accept_greedy(s["logits"], t["parent"], t["token"], s["path"], s["n_acc"], s["bonus"], None, s["ws_acc"])
    btv.btv_kv_commit(s["K"], s["V"], c["L"], c["N"], s["path"], s["n_acc"], s["new_len"])


def _prepare_attn(c, g):
    layers, L, N, Hq, Hkv, D = (c[k] for k in ("layers", "L", "N", "Hq", "Hkv", "D"))
    K, V = _kv(g, (layers, L + N, Hkv, D), c["kv"]), _kv(g, (layers, L + N, Hkv, D), c["kv"])
    Q = _randn(g, (layers, N, Hq, D), BF16)
    O = torch.zeros_like(Q)
    parent = torch.from_numpy(synth.tree_parents(g.initial_seed() % 65536, N, c["tree"])).cuda()
    size = (btv.btv_tree_verify_attn_fp8kv_workspace(N, L, Hq, Hkv, D) if c["kv"] == "fp8"
            else btv.btv_tree_verify_attn_workspace(N, L, Hq, Hkv, D, btv.BTV_BF16))
    return {"c": c, "parent": parent, "per_layer": [(Q[i], K[i], V[i], O[i]) for i in range(layers)], "out": {"O": O},
            "ws": btv.alloc_workspace(size)}


def _run_attn(s):
    L, parent, ws = s["c"]["L"], s["parent"], s["ws"]
    if s["c"]["kv"] == "fp8":
        for Q, K, V, O in s["per_layer"]:
            btv.btv_tree_verify_attn_fp8kv(Q, K, V, FP8_SCALE, FP8_SCALE, parent, L, O, ws)
    else:
        for Q, K, V, O in s["per_layer"]:
            btv.btv_tree_verify_attn(Q, K, V, parent, L, O, ws)


def _prepare_batch(c, g):
    layers, Hq, Hkv, D, B, V, nb = (c[k] for k in ("layers", "Hq", "Hkv", "D", "B", "V", "requests"))
    Ls, Ns = _lengths(c)
    table, blocks = synth.paged_layout(g.initial_seed() % 65536, [l + n for l, n in zip(Ls, Ns)])
    offsets = [0]
    for n in Ns:
        offsets.append(offsets[-1] + n)
    total, M_max, L_max = offsets[-1], max(Ns), max(Ls)
    s = {"c": c, "M_max": M_max, "L_max": L_max, "marg": _marginals(g, (nb, B, V), "sigma3"),
         "n_nodes": torch.tensor(Ns, dtype=I32, device="cuda"), "q_offset": torch.tensor(offsets, dtype=I32, device="cuda"),
         "prefix": torch.tensor(Ls, dtype=I32, device="cuda"), "table": torch.from_numpy(table).clamp(min=0).cuda(),
         "K": _kv(g, (layers, blocks, btv.BTV_PAGE, Hkv, D), c["kv"]), "V": _kv(g, (layers, blocks, btv.BTV_PAGE, Hkv, D), c["kv"]),
         "Q": _randn(g, (layers, total, Hq, D), BF16), "path": _zeros(total), "n_acc": _zeros(nb), "bonus": _zeros(nb), "new_len": _zeros(nb),
         "tree": {**_tree_out(total), "n_out": _zeros(nb), "ahat": _zeros(nb, F32)},
         "ws_build": btv.alloc_workspace(btv.btv_tree_build_batch_workspace(nb, B, V, M_max)),
         "ws_attn": btv.alloc_workspace((btv.btv_tree_verify_attn_paged_fp8kv_workspace if c["kv"] == "fp8" else
                                         btv.btv_tree_verify_attn_paged_workspace)(nb, M_max, L_max, Hq, Hkv, D)),
         "ws_acc": btv.alloc_workspace(btv.btv_tree_accept_batch_workspace(nb, total, V))}
    t = s["tree"]
    btv.btv_tree_build_batch(s["marg"], s["n_nodes"], s["q_offset"], M_max, t["parent"], t["token"], t["depth"], t["rho"], t["n_out"],
                             t["ahat"], s["ws_build"])
    best, depth = s["marg"].argmax(2), t["depth"].long().clamp(max=B - 1)
    rows = [torch.cat([best[r, :1], best[r][depth[offsets[r]:offsets[r + 1]]]]) for r in range(nb)]
    s["logits"] = _target_logits(g, torch.cat(rows), V, BF16)
    s["O"] = torch.zeros_like(s["Q"])
    s["per_layer"] = [(s["Q"][i], s["K"][i], s["V"][i], s["O"][i]) for i in range(layers)]
    s["out"] = {**t, **{k: s[k] for k in ("O", "path", "n_acc", "bonus", "new_len", "K", "V")}}
    return s


def _run_batch(s):
    c, t = s["c"], s["tree"]
    qo, M_max, L_max, table, prefix, ws = (s[k] for k in ("q_offset", "M_max", "L_max", "table", "prefix", "ws_attn"))
    btv.btv_tree_build_batch(s["marg"], s["n_nodes"], qo, M_max, t["parent"], t["token"], t["depth"], t["rho"], t["n_out"], t["ahat"],
                             s["ws_build"])
    for Q, K, V, O in s["per_layer"]:
        if c["kv"] == "fp8":
            btv.btv_tree_verify_attn_paged_fp8kv(Q, K, V, FP8_SCALE, FP8_SCALE, table, qo, prefix, t["parent"], M_max, L_max, O, ws)
        else:
            btv.btv_tree_verify_attn_paged(Q, K, V, table, qo, prefix, t["parent"], M_max, L_max, O, ws)
    btv.btv_tree_accept_greedy_batch(s["logits"], t["parent"], t["token"], qo, M_max, s["path"], s["n_acc"], s["bonus"], None, s["ws_acc"])
    btv.btv_kv_commit_paged(s["K"], s["V"], table, prefix, s["path"], s["n_acc"], s["new_len"], None, qo, M_max)


def _prepare_stochastic(c, g):
    """noise < 0: the target's logits are |noise| * N(0,1), whatever the drafter says.  noise >= 0: at a node of depth d they
    are the drafter's own log probabilities of the next position plus noise * N(0,1)."""
    N, B, V = c["N"], c["B"], c["V"]
    marg = _marginals(g, (B, V), c["marg"])
    t = _tree(marg, N)
    x = torch.randn((N + 1, V), generator=g, dtype=F32, device="cuda") * abs(c["noise"])
    if c["noise"] >= 0:
        x += marg.clamp(min=1e-30).log()[torch.cat([_zeros(1), t["depth"]]).clamp(max=B - 1).long()]
    out = {"path": _zeros(N), "n_acc": _zeros(1), "bonus": _zeros(1)}
    return {"c": c, "marg": marg, "tree": t, "logits": x.to(F32 if c["dtype"] == "fp32" else BF16), "out": out,
            "uniforms": torch.rand(N + 1, generator=g, dtype=F32, device="cuda"),
            "ws": btv.alloc_workspace(btv.btv_tree_accept_workspace(N, V, True))}


def _run_stochastic(s):
    o = s["out"]
    btv.btv_tree_accept_stochastic(s["logits"], s["marg"], s["tree"]["parent"], s["tree"]["token"], s["uniforms"], o["path"], o["n_acc"],
                                   o["bonus"], s["ws"])


def _prepare_lm_head(c, g):
    N, h, V = c["N"], c["h"], c["V"]
    W = torch.empty((V, h), dtype=BF16, device="cuda")
    for v0 in range(0, V, 16384):
        W[v0:v0 + 16384] = torch.randn((min(16384, V - v0), h), generator=g, dtype=F32, device="cuda").mul_(h ** -0.5)
    hidden = torch.randn((N + 1, h), generator=g, dtype=F32, device="cuda")
    parent = synth.tree_parents(g.initial_seed() % 65536, N, "random")
    token = torch.from_numpy(synth.sibling_distinct_tokens(g.initial_seed() % 65536, parent, V)).cuda()
    parent = torch.from_numpy(parent).cuda()
    # the target follows the tree's first nodes: the hidden state at a node's parent is turned towards its token's row
    for i in range(min(N, 4)):
        w = W[token[i].long()].float()
        hidden[parent[i].long() + 1] += 12.0 * w
    out = {"path": _zeros(N), "n_acc": _zeros(1), "bonus": _zeros(1), "argmax": _zeros(N + 1)}
    return {"c": c, "hidden": hidden.to(BF16), "W": W, "parent": parent, "token": token, "out": out,
            "ws": btv.alloc_workspace(btv.btv_tree_accept_lm_head_workspace(N, V))}


def _run_lm_head(s):
    o = s["out"]
    btv.btv_tree_accept_greedy_lm_head(s["hidden"], s["W"], s["parent"], s["token"], o["path"], o["n_acc"], o["bonus"], o["argmax"], s["ws"])


def _prepare_build(c, g):
    N, B, V = c["N"], c["B"], c["V"]
    s = {"c": c, "marg": _marginals(g, (B, V), c["marg"]), "out": _tree_out(N), "ws": btv.alloc_workspace(btv.btv_tree_build_workspace(B, V, N))}
    if c["adaptive"]:
        # 8B-shaped target at an 8k context on this GPU's nominal rates, a drafter of a tenth of a step
        model = (8192, 32, 4096, 32, 8, 128, 14336, VOCAB, 2, 2.5e15, 8e12)
        s["L_AR"] = btv.btv_verify_cost(1, *model)["latency_s"]
        s["cost"] = torch.tensor(btv.btv_verify_cost_curve(N, *model, t_other=0.1 * s["L_AR"] + 1e-4), dtype=torch.float64, device="cuda")
        s["out"]["s_best"] = _zeros(1, torch.float64)
    return s


def _run_build(s):
    o, N = s["out"], s["c"]["N"]
    if s["c"]["adaptive"]:
        btv.btv_tree_build_adaptive(s["marg"], N, s["cost"], s["L_AR"], o["parent"], o["token"], o["depth"], o["rho"], o["n_out"], o["ahat"],
                                    o["s_best"], s["ws"])
    else:
        btv.btv_tree_build(s["marg"], N, o["parent"], o["token"], o["depth"], o["rho"], o["n_out"], o["ahat"], s["ws"])


_PREPARE = {"step": _prepare_step, "attn": _prepare_attn, "batch": _prepare_batch, "stochastic": _prepare_stochastic, "lm_head": _prepare_lm_head,
            "build": _prepare_build}
_RUN = {"step": _run_step, "attn": _run_attn, "batch": _run_batch, "stochastic": _run_stochastic, "lm_head": _run_lm_head, "build": _run_build}


def prepare(case, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return _PREPARE[case["kind"]](case, g)


def run(state):
    if "graph" in state:
        state["graph"].replay()
    else:
        _RUN[state["c"]["kind"]](state)
    return state["out"]


# ----------------------------------------------------------------------------------------------------------------------
# what a pass cannot do without
# ----------------------------------------------------------------------------------------------------------------------

def _attn_work(L, N, Hq, Hkv, D, e_kv, e=2):
    """K and V once, Q and O once; a node attends to the prefix and (at least) itself."""
    return 2 * (L + N) * Hkv * D * e_kv + 2 * N * Hq * D * e + 4 * N, 4 * Hq * D * N * (L + 1)


def work(case):
    c, kind = case, case["kind"]
    if kind == "attn":
        b, f = _attn_work(c["L"], c["N"], c["Hq"], c["Hkv"], c["D"], 1 if c["kv"] == "fp8" else 2)
        return {"bytes": c["layers"] * b, "flops": c["layers"] * f}
    if kind == "step":
        e = 4 if c["dtype"] == "fp32" else 2
        b, f = _attn_work(c["L"], c["N"], c["Hq"], c["Hkv"], c["D"], e, e)
        return {"bytes": 4 * c["B"] * c["V"] + c["layers"] * b + e * (c["N"] + 1) * c["V"] + 16 * c["N"], "flops": c["layers"] * f}
    if kind == "batch":
        Ls, Ns = _lengths(c)
        per = [_attn_work(l, n, c["Hq"], c["Hkv"], c["D"], 1 if c["kv"] == "fp8" else 2) for l, n in zip(Ls, Ns)]
        b, f = (c["layers"] * sum(x[i] for x in per) for i in (0, 1))
        return {"bytes": b + 4 * c["requests"] * c["B"] * c["V"] + 2 * (sum(Ns) + len(Ns)) * c["V"] + 16 * sum(Ns), "flops": f}
    if kind == "stochastic":        # the root's row of logits and of marginals; a walk that goes deeper reads more
        return {"bytes": c["V"] * ((4 if c["dtype"] == "fp32" else 2) + 4), "flops": 4 * c["V"]}
    if kind == "lm_head":
        return {"bytes": 2 * c["h"] * (c["V"] + c["N"] + 1), "flops": 2 * (c["N"] + 1) * c["h"] * c["V"]}
    return {"bytes": 4 * c["B"] * c["V"] + 16 * c["N"], "flops": c["B"] * c["V"]}


def tolerance(case):
    kind = case["kind"]
    if kind == "build" or (kind == "step" and case["dtype"] == "fp32"):
        return {"rel": 1e-5}        # fp32 path scores and their sum; fp32 attention.  Whole numbers are exact
    if kind in ("stochastic", "lm_head"):
        return "exact"
    return {"rel": 1e-2}            # bf16 outputs; trees, tokens and paths are exact
