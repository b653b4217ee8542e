"""Timed cases: the attention work of a serving step, through the package's public entry points.

A serving engine calls this library once per layer and step: kv_cache_append
and the paged decode (PagedDecoder) for sequences that generate, and
chunked_prefill_attention for prompts.  The listed cases are those calls at
the shapes of the dual-pool deployment this library is built for (a
Llama-3-70B layer with 64 query / 8 KV heads and a bf16 cache, a
Qwen3-235B-A22B layer with 64 / 4 heads and an e4m3 cache, pools with
C_max 8K and 64K) and at the small, ragged and lightly loaded ends of the
same ranges; draw() gives more of them.  The host calls (pool, router, cost
model) take well under a microsecond per request and are not on this path.

A case is a dict of plain values:
  kind       "decode", "step" (append, then decode), "append" or "prefill"
  layers     layers one pass runs, each with a cache and buffers of its own
             (the same context lengths and block tables, as in a model)
  batch, hq, hkv, c_max, num_blocks, fp8, out_fp32
  lens       how context lengths are drawn (see lengths()), or the lengths
             themselves as text "2048,8192"
  lens_seed  seed of that draw: lengths belong to the case, values to `seed`
  chunk      prefill only: query tokens of each sequence's chunk (the last
             ones of its context); 0: the whole context is one fresh prompt
"""
import math

import numpy as np
import torch

from paper_2604_08075_amd import binding

BLOCK = 16
DIM = 128
SCALE = 1.0 / math.sqrt(DIM)
E4M3_MAX = 448.0

LLAMA = dict(hq=64, hkv=8, fp8=False, num_blocks=49152)
QWEN = dict(hq=64, hkv=4, fp8=True, num_blocks=167936)


def _case(name, kind, lens, batch, c_max, layers=1, lens_seed=0, out_fp32=False, chunk=0, **model):
    return dict(name=name, kind=kind, lens=lens, batch=batch, c_max=c_max, layers=layers, lens_seed=lens_seed,
                out_fp32=out_fp32, chunk=chunk, **model)


def listed():
    return [
        # A handful of short chats on a small model: every kernel is a few
        # microseconds long, latency and launches are all there is.
        _case("step_tiny_bf16", "step", "uniform", 4, 512, layers=4, lens_seed=1, out_fp32=True, hq=8, hkv=2,
              fp8=False, num_blocks=512),
        # The short pool at its full batch: the ordinary decode step.
        _case("decode_short_bf16", "decode", "lognormal", 128, 8192, layers=2, lens_seed=2, **LLAMA),
        # The long pool: few sequences, contexts of 8K to 64K.
        _case("decode_long_bf16", "decode", "pareto", 16, 65536, layers=2, lens_seed=3, **LLAMA),
        # A homogeneous pool (what the router replaces): few sequences, one or
        # two of them long.  Six layers, so that the step streams from memory.
        _case("decode_mixed_bf16", "decode", "mixture", 16, 65536, layers=6, lens_seed=4, **LLAMA),
        # The short pool of the fp8 deployment, GQA 16.
        _case("decode_short_fp8", "decode", "lognormal", 256, 8192, layers=3, lens_seed=5, **QWEN),
        # The same pool at a quiet hour: an odd, small batch (twelve layers, to
        # stream from memory too).
        _case("decode_quiet_fp8", "decode", "lognormal", 13, 8192, layers=12, lens_seed=6,
              **dict(QWEN, num_blocks=32768)),
        # Every sequence's new token written into its page, fp8 encoding.
        _case("append_fp8", "append", "uniform", 256, 128, layers=4, lens_seed=7, hq=64, hkv=4, fp8=True,
              num_blocks=2048),
        # Chunks of the default size (2,048 tokens) of four long prompts.
        _case("prefill_chunks_bf16", "prefill", "2048,8192,16384,32768", 4, 32768, chunk=2048, **LLAMA),
        # Chunks of a short pool's longest prompts, fp8 cache.
        _case("prefill_chunks_fp8", "prefill", "2048,4096,6144,8192", 4, 8192, chunk=2048, **QWEN),
        # A round of ordinary fresh prompts of ragged lengths.
        _case("prefill_prompts_bf16", "prefill", "lognormal", 11, 8192, lens_seed=8, **LLAMA),
        # The last, part-filled chunk of one long prompt, alone in its round.
        _case("prefill_lastchunk_bf16", "prefill", "20861", 1, 65536, chunk=381, **LLAMA),
        # Short prompts on a small model with GQA 4, e4m3 cache.
        _case("prefill_small_fp8", "prefill", "uniform", 3, 512, lens_seed=9, hq=8, hkv=2, fp8=True, num_blocks=512),
    ]


def lengths(case):
    """Context lengths (cached tokens, the new ones included), int64 [batch]."""
    if "," in case["lens"] or case["lens"].isdigit():
        return np.array([int(x) for x in case["lens"].split(",")], dtype=np.int64)
    rng = np.random.default_rng(case["lens_seed"])
    n, c_max = case["batch"], case["c_max"]

    def lognormal():  # prompts of median 600 tokens and up to 428 generated ones
        prompt = np.clip(np.rint(rng.lognormal(math.log(600.0), 1.2, n)), 16, 8192)
        return np.minimum(prompt + rng.integers(1, 429, n), min(c_max, 8192)).astype(np.int64)

    def pareto():  # alpha 1.5 between 8,192 tokens and c_max
        u = rng.random(n)
        return np.floor(8192 / (1.0 - u * (1.0 - (8192 / c_max) ** 1.5)) ** (1 / 1.5)).astype(np.int64).clip(1, c_max)

    if case["lens"] == "uniform":
        return rng.integers(1, c_max + 1, n).astype(np.int64)
    if case["lens"] == "lognormal":
        return lognormal()
    if case["lens"] == "pareto":
        return pareto()
    is_long = rng.random(n) < 0.15  # "mixture"
    return np.where(is_long, pareto(), lognormal())


def chunks(case):
    """Query tokens of each sequence (prefill), int64 [batch]."""
    ctx = lengths(case)
    return np.minimum(case["chunk"], ctx) if case["chunk"] else ctx


def work(case):
    ctx, eb = lengths(case), 1 if case["fp8"] else 2
    hq, hkv, b, layers = case["hq"], case["hkv"], case["batch"], case["layers"]
    out_b = 4 if case["out_fp32"] else 2
    kv_token = hkv * DIM * 2  # K and V values of one token
    if case["kind"] == "prefill":
        n = chunks(case)
        pairs = int((n * ctx - n * (n - 1) // 2).sum())
        flops = 4 * DIM * hq * pairs
        nbytes = int(ctx.sum()) * kv_token * eb + int(n.sum()) * hq * DIM * (2 + out_b)
    else:
        flops = nbytes = 0
        if case["kind"] != "append":
            flops += 4 * DIM * hq * int(ctx.sum())
            nbytes += int(ctx.sum()) * kv_token * eb + b * hq * DIM * (2 + out_b)
        if case["kind"] != "decode":
            nbytes += b * kv_token * (2 + eb)
    return {"bytes": nbytes * layers, "flops": flops * layers}


def draw(rng):
    most = max((work(c) for c in listed() if c["kind"] == "prefill"), key=lambda x: x["flops"])["flops"]
    most_bytes = max(work(c)["bytes"] for c in listed())
    while True:
        kind = rng.choice(["decode", "decode", "decode", "step", "append", "prefill", "prefill", "prefill"])
        hkv = rng.choice([1, 2, 3, 4, 8, 8])
        group = rng.choice([1, 2, 4, 5, 7, 8, 8, 12, 16, 16])
        c = _case("", kind, rng.choice(["uniform", "lognormal"]), 1, 0, lens_seed=rng.randrange(1 << 30),
                  out_fp32=rng.random() < 0.25, hkv=hkv, hq=hkv * group, fp8=rng.random() < 0.5)
        del c["name"]
        if kind == "prefill":
            c["batch"] = round(math.exp(rng.uniform(0, math.log(24))))
            c["c_max"] = round(math.exp(rng.uniform(math.log(64), math.log(32768))))
            if rng.random() < 0.5:
                c["chunk"] = round(math.exp(rng.uniform(math.log(16), math.log(2048))))
        else:
            c["batch"] = round(math.exp(rng.uniform(0, math.log(512))))
            c["c_max"] = round(math.exp(rng.uniform(math.log(64), math.log(65536))))
            if c["c_max"] > 16384 and rng.random() < 0.7:
                c["lens"] = rng.choice(["pareto", "mixture"])
            c["layers"] = rng.choice([1, 2, 4])
            if kind != "decode":  # the cache is an output: a pool of small pages' worth
                c["c_max"] = min(c["c_max"], 512)
                c["batch"] = min(c["batch"], 256)
                c["lens"] = "uniform"
        if c["lens"] == "lognormal" and c["c_max"] < 2048:
            c["lens"] = "uniform"
        used = int((-(-lengths(c) // BLOCK)).sum())
        c["num_blocks"] = min(max(2 * used, 64), 167936)
        if kind == "step" or kind == "append":
            c["num_blocks"] = used + 1 + used // 8
        size = c["num_blocks"] * hkv * BLOCK * DIM * 2 * (1 if c["fp8"] else 2) * c["layers"]
        w = work(c)
        if used <= c["num_blocks"] and size <= 24e9 and w["flops"] <= most and w["bytes"] <= most_bytes:
            if kind not in ("step", "append") or size <= 128e6:
                return c


def _inputs(case, seed):
    """Every input of the pass, on the GPU, from the seed alone."""
    dev = torch.device("cuda")
    g = torch.Generator(device=dev).manual_seed(seed)
    ctx = lengths(case)
    b, hq, hkv, nb = case["batch"], case["hq"], case["hkv"], case["num_blocks"]
    max_blocks = -(-case["c_max"] // BLOCK)
    # pages scattered over the pool, -1 past each sequence's own
    perm = np.random.default_rng(seed).permutation(nb).astype(np.int32)
    tables = np.full((b, max_blocks), -1, dtype=np.int32)
    at = 0
    for s, t in enumerate(ctx):
        n = -(-int(t) // BLOCK)
        tables[s, :n] = perm[at:at + n]
        at += n
    x = dict(tables=torch.from_numpy(tables).to(dev), ctx=torch.from_numpy(ctx.astype(np.int32)).to(dev),
             ks=None, vs=None, layers=[])
    if case["fp8"]:  # per-head scales of an amax near 4.5 standard deviations
        x["ks"], x["vs"] = ((4.5 + torch.rand(hkv, generator=g, device=dev)) / E4M3_MAX for _ in range(2))
    rows = b
    if case["kind"] == "prefill":
        n = chunks(case)
        rows = int(n.sum())
        x["q_start"] = torch.from_numpy(np.concatenate([[0], np.cumsum(n)]).astype(np.int32)).to(dev)

    def normal(*shape):
        return torch.randn(shape, generator=g, device=dev, dtype=torch.bfloat16)

    def cache(*shape):
        if not case["fp8"]:
            return normal(*shape)
        t = torch.empty(shape, dtype=torch.uint8, device=dev)
        for i in range(0, nb, 8192):  # unit-variance values over a scale of 1 / 93, saturating
            part = torch.randn((min(8192, nb - i),) + shape[1:], generator=g, device=dev) * 93.0
            t[i:i + 8192] = part.clamp_(-E4M3_MAX, E4M3_MAX).to(torch.float8_e4m3fn).view(torch.uint8)
        return t

    for _ in range(case["layers"]):
        layer = dict(k=cache(nb, hkv, BLOCK, DIM), v=cache(nb, hkv, DIM, BLOCK))
        if case["kind"] != "append":
            layer["q"] = normal(rows, hq, DIM)
        if case["kind"] in ("step", "append"):
            layer["k_new"], layer["v_new"] = normal(b, hkv, DIM), normal(b, hkv, DIM)
        x["layers"].append(layer)
    if case["kind"] in ("step", "append"):
        x["pos"] = (x["ctx"] - 1).contiguous()
    return x


def prepare(case, seed):
    x = _inputs(case, seed)
    x["case"] = case
    max_blocks = x["tables"].shape[1]
    b, hq, hkv, nb, c_max = case["batch"], case["hq"], case["hkv"], case["num_blocks"], case["c_max"]
    odt = torch.float32 if case["out_fp32"] else torch.bfloat16
    if case["kind"] == "prefill":
        rows = x["layers"][0]["q"].shape[0]
        x["shape"] = binding.prefill_shape(b, hq, hkv, max_blocks, c_max, nb, rows, kv_fp8=case["fp8"],
                                           out_fp32=case["out_fp32"])
        for layer in x["layers"]:
            layer["out"] = torch.zeros((rows, hq, DIM), dtype=odt, device="cuda")
        return x
    # one decoder (and its workspace) serves every layer of the step
    x["decoder"] = binding.PagedDecoder(b, hq, hkv, max_blocks, c_max, nb, kv_fp8=case["fp8"],
                                        out_fp32=case["out_fp32"])
    if case["kind"] != "append":
        for layer in x["layers"]:
            layer["out"] = x["decoder"].new_out()
    return x


def run(x):
    kind = x["case"]["kind"]
    outs = []
    for layer in x["layers"]:
        if kind == "prefill":
            binding.chunked_prefill_attention(layer["q"], layer["k"], layer["v"], x["tables"], x["ctx"],
                                              x["q_start"], SCALE, layer["out"], x["shape"], x["ks"], x["vs"])
            outs.append(layer["out"])
            continue
        if kind != "decode":
            binding.kv_cache_append(layer["k_new"], layer["v_new"], layer["k"], layer["v"], x["tables"], x["pos"],
                                    x["decoder"].shape, x["ks"], x["vs"])
            outs += [layer["k"], layer["v"]]
        if kind != "append":
            x["decoder"](layer["q"], layer["k"], layer["v"], x["tables"], x["ctx"], SCALE, layer["out"], x["ks"],
                         x["vs"])
            outs.append(layer["out"])
    return outs


def tolerance(case):
    # Appends move or encode single values: the cache must match bit for bit.
    if case["kind"] == "append":
        return "exact"
    # Probabilities enter the second product as bf16 (2^-9 relative each) and
    # bf16 outputs are rounded once more.  Measured against exact(): 0.8e-3 to
    # 2.4e-3 by norm; about four times that.
    return {"rel": 8e-3, "max": 0.1}


def exact(case, seed):
    x = _inputs(case, seed)
    ctx, hq, hkv = lengths(case), case["hq"], case["hkv"]
    group = hq // hkv
    n_new = chunks(case) if case["kind"] == "prefill" else np.ones(case["batch"], dtype=np.int64)
    outs = []
    for layer in x["layers"]:
        k_all, v_all = layer["k"], layer["v"]
        if case["kind"] in ("step", "append"):  # the new token's row and column
            pos = x["pos"].long()
            blk = x["tables"].long().gather(1, (pos // BLOCK)[:, None])[:, 0]
            if case["fp8"]:
                enc = [(layer[n].float() / s[:, None]).clamp(-E4M3_MAX, E4M3_MAX).to(torch.float8_e4m3fn)
                       .view(torch.uint8) for n, s in (("k_new", x["ks"]), ("v_new", x["vs"]))]
            else:
                enc = [layer["k_new"], layer["v_new"]]
            k_all[blk, :, pos % BLOCK] = enc[0]
            v_all[blk, :, :, pos % BLOCK] = enc[1]
            outs += [k_all, v_all] if case["fp8"] else [k_all.double(), v_all.double()]
            if case["kind"] == "append":
                continue
        out = torch.empty(layer["q"].shape, dtype=torch.float64, device=layer["q"].device)
        row = 0
        for s, (t, n) in enumerate(zip(ctx.tolist(), n_new.tolist())):
            ids = x["tables"][s, :-(-t // BLOCK)].long()
            if case["fp8"]:
                k, v = (a[ids].view(torch.float8_e4m3fn).double() for a in (k_all, v_all))
                k, v = k * x["ks"].double()[:, None, None], v * x["vs"].double()[:, None, None]
            else:
                k, v = k_all[ids].double(), v_all[ids].double()
            k = k.permute(1, 0, 2, 3).reshape(hkv, -1, DIM)[:, :t]
            v = v.permute(1, 0, 3, 2).reshape(hkv, -1, DIM)[:, :t]
            future = None
            if n > 1:
                future = torch.arange(t, device=k.device)[None, :] > torch.arange(t - n, t, device=k.device)[:, None]
            for h in range(hq):
                z = (layer["q"][row:row + n, h].double() * SCALE) @ k[h // group].t()
                if future is not None:
                    z.masked_fill_(future, -math.inf)
                out[row:row + n, h] = torch.softmax(z, dim=-1) @ v[h // group]
            row += n
        outs.append(out)
    return outs
