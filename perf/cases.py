"""The work whose time matters to a user of this library, as cases that a timing program can prepare and run.

A case names what is called ("op") and the shape of the batch it is called on:

  decode      one decode step over a packed cache, called eagerly as a serving loop does
  stack       one decode step of a whole model: a cache per layer, the per-layer calls replayed from a HIP graph
  bf16        the same decode step over the uncompressed bf16 cache
  compress    the one-shot pass after prefill (rdkv_compress), and the first decode step on its cache
  stages      the same pass through the staged entry points, for a caller that keeps weights and bit maps
  request     the life of one request in one layer: compress the prompt, append and decode token by token, compress the
              appended tokens, decode once more

Shapes are those of paper_2605_08317_amd/workloads.py (8B- and 70B-shaped layers, head_dim 128) and their neighbours;
tensors are synthetic, with that file's recipe: normal K and V, a few key channels ten times larger, and for long
contexts attention sinks that the queries look at.
"""
import math
import random

import torch

from paper_2605_08317_amd import binding as b

D = 128

#: Distortion tables for tier subsets: all widths (the library's default), and keep / 4 bit / evict.
TIERS = {
    "all": {},
    "tri": {"tiers": (0, 4, 16), "eps_v": (1.0, 0.0140, 0.0), "eps_k": (1.0, 0.0140, 0.0)},
}


def _case(op, name=None, *, batch=1, hq=32, hkv=8, lo, hi=None, budgets="1", mode="token", tiers="all", per_channel=False,
          group=32, s_obs=32, sinks=False, layers=1, tokens=0, pareto=False):
    c = {"op": op, "batch": batch, "hq": hq, "hkv": hkv, "lo": lo, "hi": hi or lo, "budgets": budgets, "mode": mode,
         "tiers": tiers, "per_channel": per_channel, "group": group, "s_obs": s_obs, "sinks": sinks, "layers": layers,
         "tokens": tokens, "pareto": pareto}
    return dict(c, name=name) if name else c


def listed():
    return [
        # The smallest call there is in earnest: two KV heads of a tensor-parallel shard, 4K context.  Launch latency
        # and the host side of the call.
        _case("decode", "decode_tiny", hq=8, hkv=2, lo=4096, budgets="2"),
        # A model's decode step at long context, as served: 32 layers, one graph.
        _case("stack", "stack_128k", lo=131072, budgets="0.4", s_obs=64, sinks=True, layers=32),
        # Batched serving of a 70B-shaped layer: ragged contexts, a budget per sequence, 8 query heads per KV head.
        _case("decode", "decode_batch_70b", batch=16, hq=64, lo=8192, hi=32768, budgets="0.5,1,2,4"),
        # Long contexts at a budget that keeps quality close to bf16: keep / 4 bit / evict, one scale per row, ragged.
        _case("decode", "decode_tri_long", batch=4, lo=90001, hi=131072, budgets="4,8", tiers="tri", group=128, sinks=True),
        # Keys channel by channel (the paper's own arrangement): one 64K sequence with heavy-tailed weights.
        _case("decode", "decode_mixed_64k", lo=65536, budgets="1", mode="channel", pareto=True),
        # The same for a batch, with the paper's one scale per key channel.
        _case("decode", "decode_mixed_batch", batch=16, lo=65536, budgets="1", mode="channel", per_channel=True, pareto=True),
        # The uncompressed path that everything is compared with, at the same context as the stack.
        _case("bf16", "bf16_128k", lo=131072, sinks=True),
        # Compression of a short prompt: a pass of small kernels.
        _case("compress", "compress_tiny", hq=8, hkv=2, lo=4096, budgets="2"),
        # Compression of one layer of a long prompt.
        _case("compress", "compress_128k", lo=131072, budgets="0.4", s_obs=64, sinks=True),
        # Compression of a ragged batch of a 70B-shaped layer.
        _case("compress", "compress_batch_70b", batch=16, hq=64, lo=8192, hi=32768, budgets="0.5,1,2,4"),
        # Channel-wise keys through the staged calls, a length that is no multiple of any tile.
        _case("stages", "stages_mixed_50k", lo=50021, budgets="1", mode="channel"),
        # One layer's share of a request: prompt, 64 generated tokens, the generated tokens compressed.
        _case("request", "request_8b", lo=32768, budgets="1", tokens=64),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["decode", "decode", "decode", "stack", "bf16", "compress", "compress", "stages", "request"])
    hkv = rng.choice([2, 4, 8])
    g = rng.choice([1, 2, 4, 4, 4, 8, 8])
    kw = {"hkv": hkv, "hq": hkv * g, "s_obs": rng.choice([32, 64]), "sinks": rng.random() < 0.5}
    kw["batch"] = 1 if op in ("stack", "request") else _log(rng, 1, 16)
    longest = 32768 if op == "request" else 131072
    if kw["batch"] > 4:
        longest = 32768           # what the largest listed batches hold
    if op in ("compress", "stages"):   # window rows times tokens: at most what the largest listed pass has
        longest = min(longest, 600_000_000 // (kw["batch"] * hkv * g * kw["s_obs"]))
    hi = _log(rng, 512, longest)
    kw["hi"] = hi
    kw["lo"] = hi if kw["batch"] == 1 else max(256, int(hi * rng.uniform(0.25, 1.0)))
    budgets = ["%.3g" % math.exp(rng.uniform(math.log(0.4), math.log(8.0))) for _ in range(rng.choice([1, 1, 3]))]
    if op == "bf16":
        return _case(op, lo=kw["lo"], hi=hi, batch=kw["batch"], hkv=hkv, hq=hkv * g, sinks=kw["sinks"])
    if rng.random() < (1.0 if op == "stages" else 0.3):
        kw.update(mode="channel", per_channel=rng.random() < 0.5, pareto=op == "decode" and rng.random() < 0.5)
    else:
        kw.update(tiers=rng.choice(["all", "all", "tri"]))
    kw["group"] = rng.choice([32, 32, 128])
    if op == "stack":
        kw["layers"] = rng.choice([2, 8, 16])
        budgets = [x if float(x) < 2 else "2" for x in budgets]
    if op == "request":
        kw["tokens"] = rng.randint(kw["s_obs"], 80)
    return _case(op, budgets=",".join(budgets), **kw)


def _lens(case):
    """Context length of every sequence: part of the case, the same for every seed."""
    if case["lo"] == case["hi"]:
        return [case["hi"]] * case["batch"]
    rng = random.Random("%d %d %d" % (case["batch"], case["lo"], case["hi"]))
    return [case["hi"]] + [rng.randint(case["lo"], case["hi"]) for _ in range(case["batch"] - 1)]


def _budgets(case):
    x = [float(v) for v in case["budgets"].split(",")]
    return [x[i % len(x)] for i in range(case["batch"])]


def _config(case, seq_lens, budgets):
    """As a PyTorch program makes it: device memory comes from PyTorch's caching allocator."""
    return b.Config(seq_lens, case["hq"], case["hkv"], budget_bits=budgets, s_obs=case["s_obs"], group_size=case["group"],
                    k_mode=b.RDKV_K_CHANNELWISE if case["mode"] == "channel" else b.RDKV_K_TOKENWISE,
                    k_scale_per_channel=int(case["per_channel"]), **TIERS[case["tiers"]], **b.torch_allocator_hooks())


def _inputs(case, gen):
    """K, V (flat, a block [hkv][T][128] per sequence), the window queries and a decode query of one layer."""
    lens, hq, hkv = _lens(case), case["hq"], case["hkv"]
    g = hq // hkv

    def normal(*shape):
        return torch.randn(shape, generator=gen, device="cuda", dtype=torch.bfloat16)

    total = sum(lens) * hkv * D
    K, V = torch.empty(total, device="cuda", dtype=torch.bfloat16), normal(total)
    q_obs, q = normal(case["batch"], hq, case["s_obs"], D), normal(case["batch"], hq, D)
    at = 0
    for s, T in enumerate(lens):
        k = K[at:at + hkv * T * D].view(hkv, T, D)
        k.normal_(generator=gen)
        at += hkv * T * D
        if case["sinks"]:        # 1 % of the positions, along one direction per head, that the queries point to
            u = torch.randn((hkv, 1, D), generator=gen, device="cuda")
            u = 9.5 * u / u.norm(dim=-1, keepdim=True)
            pos = torch.randint(0, T, (max(1, T // 100),), generator=gen, device="cuda")
            k[:, pos] = (k[:, pos].float() + u).to(torch.bfloat16)
            up = u.repeat_interleave(g, 0)
            q_obs[s] = (q_obs[s].float() + up).to(torch.bfloat16)
            q[s] = (q[s].float() + up[:, 0]).to(torch.bfloat16)
        else:                    # a few key channels per head are ten times larger
            ch = torch.rand((hkv, D), generator=gen, device="cuda").topk(3, dim=-1).indices
            scale = torch.ones((hkv, 1, D), device="cuda", dtype=torch.bfloat16).scatter_(2, ch[:, None], 10.0)
            k.mul_(scale)
    return lens, K, V, q_obs, q


def _cache(case, cfg, K, V, q_obs, gen):
    """The packed cache of one layer.  pareto: heavy-tailed token weights supplied by the caller, 1 + Pareto(1.2)."""
    if not case["pareto"]:
        return b.rdkv_compress(cfg, K, V, q_obs)
    w_tok = 1.0 + torch.rand(cfg.total_tokens, generator=gen, device="cuda").clamp_(1e-7, 1.0).pow_(-1.0 / 1.2)
    w_ch = b.rdkv_weights(cfg, K, q_obs, want_channel=True)[1] if case["mode"] == "channel" else None
    return b.rdkv_pack(cfg, K, V, *b.rdkv_allocate(cfg, w_tok, w_ch))


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    op, budgets = case["op"], _budgets(case)
    st = {"case": case, "op": op}
    if op == "stack":
        st["caches"], qs = [], []
        for _ in range(case["layers"]):
            lens, K, V, q_obs, q = _inputs(case, gen)
            st["caches"].append(_cache(case, _config(case, lens, budgets), K, V, q_obs, gen))
            qs.append(q)
            del K, V
        st["q"] = torch.stack(qs)
        st["out"] = torch.empty(st["q"].shape, device="cuda", dtype=torch.float32)
        st["lse"] = torch.empty(st["q"].shape[:-1], device="cuda", dtype=torch.float32)
        torch.cuda.synchronize()
        st["graph"] = torch.cuda.CUDAGraph()
        with torch.cuda.graph(st["graph"]):
            for layer, cache in enumerate(st["caches"]):
                b.rdkv_decode_attn(cache, st["q"][layer], st["out"][layer], st["lse"][layer])
        return st
    lens, K, V, q_obs, q = _inputs(case, gen)
    cfg = _config(case, lens, budgets)
    st.update(cfg=cfg, lens=lens, q=q)
    if op == "decode":
        st["cache"] = _cache(case, cfg, K, V, q_obs, gen)
        torch.cuda.synchronize()
        return st
    st.update(K=K, V=V, q_obs=q_obs)
    if op == "bf16":
        st["workspace"] = torch.empty(max(16, b.rdkv_decode_bf16_workspace_bytes(lens, case["hq"], case["hkv"])),
                                      device="cuda", dtype=torch.uint8)
    if op == "request":
        n = case["tokens"]
        new = (n, case["batch"], case["hkv"], D)
        st["k_new"] = torch.randn(new, generator=gen, device="cuda", dtype=torch.bfloat16)
        st["v_new"] = torch.randn(new, generator=gen, device="cuda", dtype=torch.bfloat16)
        st["q_new"] = torch.randn((n + 1, case["batch"], case["hq"], D), generator=gen, device="cuda", dtype=torch.bfloat16)
        st["q_tail"] = st["q_new"][n - case["s_obs"]:n].permute(1, 2, 0, 3).contiguous()
        st["tail_cfg"] = _config(case, [n] * case["batch"], [2.0] * case["batch"])
    return st


def run(st):
    op = st["op"]
    if op == "decode":
        return b.rdkv_decode_attn(st["cache"], st["q"])
    if op == "stack":
        st["graph"].replay()
        return st["out"], st["lse"]
    case, cfg = st["case"], st["cfg"]
    if op == "bf16":
        return b.rdkv_decode_attn_bf16(st["K"], st["V"], st["lens"], case["hq"], case["hkv"], st["q"],
                                       workspace=st["workspace"])
    if op == "compress":
        cache = b.rdkv_compress(cfg, st["K"], st["V"], st["q_obs"])
        return b.rdkv_decode_attn(cache, st["q"])
    if op == "stages":
        w_tok, w_ch = b.rdkv_weights(cfg, st["K"], st["q_obs"], want_channel=case["mode"] == "channel")
        bits_tok, bits_ch = b.rdkv_allocate(cfg, w_tok, w_ch)
        cache = b.rdkv_pack(cfg, st["K"], st["V"], bits_tok, bits_ch)
        return [w_tok, w_ch, bits_tok, bits_ch, *b.rdkv_decode_attn(cache, st["q"])]
    # request
    n = case["tokens"]
    out = torch.empty(st["q_new"].shape, device="cuda", dtype=torch.float32)
    lse = torch.empty(st["q_new"].shape[:-1], device="cuda", dtype=torch.float32)
    cache = b.rdkv_compress(cfg, st["K"], st["V"], st["q_obs"])
    b.rdkv_cache_reserve_tail(cache, n)
    for i in range(n):
        b.rdkv_cache_append(cache, st["k_new"][i], st["v_new"][i])
        b.rdkv_decode_attn(cache, st["q_new"][i], out[i], lse[i])
    b.rdkv_cache_rebudget_tail(cache, st["tail_cfg"], st["q_tail"])
    b.rdkv_decode_attn(cache, st["q_new"][n], out[n], lse[n])
    return out, lse


def work(case):
    """Bytes: every input and every output once.  The packed cache counts as its codes (the budget) and 32 bytes of
    scales and offsets per kept row, with 2.5 bits as a kept row's average width; a budget over 16 bits stores bf16."""
    hkv, hq, batch, lens = case["hkv"], case["hq"], case["batch"], _lens(case)
    g = hq // hkv
    tokens = [T * hkv for T in lens]
    q_out = batch * hq * (D * (2 + 4) + 4)
    kept = [min(n, n * x / 2.5) for n, x in zip(tokens, _budgets(case))]
    packed = sum(n * min(16.0, x) * 2 * D / 8 for n, x in zip(tokens, _budgets(case))) + 32 * sum(kept)
    attend = 4 * g * D                                                # flops of a decode step per row it attends to
    if case["op"] == "bf16":
        return {"bytes": sum(tokens) * 4 * D + q_out, "flops": sum(tokens) * attend}
    if case["op"] in ("decode", "stack"):
        return {"bytes": case["layers"] * (packed + q_out), "flops": case["layers"] * sum(kept) * attend}
    # the pass reads all keys, the kept rows' values and the window queries; the cache is written and read once
    nbytes = sum(tokens) * 2 * D + sum(kept) * 2 * D + batch * hq * case["s_obs"] * D * 2 + 2 * packed + q_out
    flops = sum(tokens) * 2 * g * case["s_obs"] * D + sum(kept) * attend
    if case["op"] == "stages":
        nbytes += sum(tokens) * (2 * 4 + 3)                           # weights written and read, bit map written and read twice
    if case["op"] == "request":
        n = case["tokens"]
        nbytes += n * (packed + q_out + batch * hkv * 4 * D * 2)      # every step reads the cache again
        nbytes += (n * (n + 1) // 2) * batch * hkv * 4 * D            # and the tokens appended so far
        flops += n * sum(kept) * attend
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    if case["op"] == "bf16":
        # exact bf16 products and fp32 sums; probabilities enter P V as two bf16 terms, 16 bits together
        return {"rel": 1e-4}
    if case["op"] in ("decode", "stack"):
        # probabilities times V scales are rounded to fp16 (11 bits) before the matrix product with the codes
        return {"rel": 2e-3}
    # as above; fp32 weights may be summed in another order, so a token on a tier's threshold can go either way
    return {"rel": 4e-3, "differ": 1e-3}
