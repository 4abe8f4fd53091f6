"""Performance cases of the library: what its users call, through the Python
binding, over the sizes a serving engine meets.

A case is a dict of plain values:

  kind       "step" (the new token of every sequence written, then decode
             attention, in one call; at head sizes 64 and 256 the append
             through the page table followed by the attention call),
             "attention" (decode attention alone), "cascade" (the step over a
             shared prefix), "write" (quantize-on-write), "calibrate" (the
             sweep of the scale constant)
  cache      "fp4" (the library's cache), or a comparison cache: "fp8",
             "bf16", "tq4"
  batch, q_heads, kv_heads, head_dim
  context    every sequence's length ("spread" 0), or the median of a
             lognormal law of sigma "spread", clipped to [low, high];
             the lengths follow from "lens", their order from the seed
  bound      the host-side bound of the lengths the caller passes: 0 for the
             longest length itself, else a limit (an engine that captures its
             step in a graph passes the model's limit)
  partition  context tokens per partition, 0 for the library's default
  dtype      of queries, K and V ("float32", "bfloat16", "float16"); out: of
             the output; fp8_query: the query is cast by a call of its own
  rotate_v   V stored rotated

Keys and values are N(0, 1) with 4 outlier channels per KV head times 20 (the
recipe of the package's workloads), pages are a random permutation of the
pool.  Every state holds its own pools, page table, workspace and output, as
an engine's layer does.
"""
import math
import random

import numpy as np
import torch

from paper_2606_20474_amd import uq

PAGE = 16
C = 0.156
DTYPES = {"float32": torch.float32, "bfloat16": torch.bfloat16, "float16": torch.float16}
REF_SCALE = 0.25   # per-tensor scale of the FP8 cache: outliers of about 80 stay inside 448 * 0.25
# bytes per token and KV head of K and V together, head size 128
REF_BYTES = {"fp8": 256, "bf16": 512, "tq4": 148}
# 16 ascending key levels: the Lloyd-Max quantizer of N(0, 1) (Max, 1960) over sqrt(128)
_MAX16 = (0.1284, 0.3881, 0.6568, 0.9424, 1.2562, 1.6181, 2.0691, 2.7326)
CODEBOOK = [s * m / math.sqrt(128) for s, ms in ((-1, _MAX16[::-1]), (1, _MAX16)) for m in ms]


def _decode(name, kind, cache="fp4", batch=1, q_heads=64, kv_heads=8, head_dim=128, context=1024, spread=0.0, low=1,
            high=131072, lens=0, bound=0, partition=0, dtype="bfloat16", out="bfloat16", rotate_v=True,
            fp8_query=False, prefix=0):
    return dict(name=name, kind=kind, cache=cache, batch=batch, q_heads=q_heads, kv_heads=kv_heads,
                head_dim=head_dim, context=context, spread=spread, low=low, high=high, lens=lens, bound=bound,
                partition=partition, dtype=dtype, out=out, rotate_v=rotate_v, fp8_query=fp8_query, prefix=prefix)


def listed():
    return [
        # one user at the start of a conversation: the smallest decode step, where the launches are what counts
        _decode("step-b1-ctx1531", "step", context=1531),
        # one user with a long document: a single sequence has to fill the chip by splitting its context
        _decode("step-b1-ctx120011", "step", context=120011, rotate_v=False),
        # a small continuous batch of mixed lengths, stepped with the model's length limit as the bound
        _decode("step-b12-ragged", "step", batch=12, q_heads=48, context=8192, spread=1.0, low=256, high=65536, lens=3,
                bound=65536),
        # the Qwen3-235B-like layer of the headline benchmark, in the library's default types
        _decode("step-b32-ctx32k", "step", batch=32, kv_heads=4, context=32768, dtype="float32", out="float32"),
        # the high-concurrency layer: the largest call, one whole GPU's cache of one layer
        _decode("attention-b256-ctx128k", "attention", batch=256, context=131072, partition=4096, out="float32"),
        # the MiniMax-like layer: agent traces over a shared 16k prompt, lognormal contexts
        _decode("cascade-b64-shared16k", "cascade", batch=64, q_heads=48, context=32768, spread=0.8, low=8192,
                high=131072, lens=2, prefix=16384),
        # one of eight GPUs' share of a GPT-OSS-like layer (head size 64, one KV head), a ragged batch
        _decode("head64-b64-ragged", "step", batch=64, q_heads=8, kv_heads=1, head_dim=64, context=12288, spread=0.7,
                low=512, high=65536, lens=5),
        # a head-size-256 layer with contexts of a few thousand tokens
        _decode("head256-b16-ctx4k", "step", batch=16, q_heads=16, kv_heads=4, head_dim=256, context=4099, spread=0.3,
                low=64, high=16384, lens=6, dtype="float16", out="float32"),
        # the codebook cache of the paper's other endpoint, a middle-sized batch
        _decode("tq4-b16-ctx16k", "step", cache="tq4", batch=16, kv_heads=4, context=16384, spread=0.2, low=1024,
                high=32768, lens=7),
        # a whole prompt batch written at once: 65536 tokens of 8 KV heads into random pages
        dict(name="write-prefill-65536", kind="write", cache="fp4", tokens=65536, kv_heads=8, head_dim=128,
             dtype="bfloat16", rotate_v=True, fused=False, paged=False, padding=0),
        # an engine's chunk of about 2k tokens: K and V as views of a fused QKV buffer, some rows padding
        dict(name="write-chunk-2309", kind="write", cache="fp4", tokens=2309, kv_heads=4, head_dim=128,
             dtype="bfloat16", rotate_v=True, fused=True, paged=True, padding=37),
        # the offline fit of c on captured key rows: one sweep of 46 constants
        dict(name="calibrate-131072x46", kind="calibrate", rows=131072, constants=46, dtype="float32", rotate=True,
             pow2=True),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "step", "step", "attention", "cascade", "head", "head", "ref", "write", "write",
                       "calibrate"])
    if kind == "write":
        return dict(kind="write", cache=rng.choice(["fp4", "fp4", "fp4", "fp8", "tq4"]), tokens=_log(rng, 1, 65536),
                    kv_heads=rng.choice([1, 2, 3, 4, 8]), head_dim=128, dtype=rng.choice(list(DTYPES)),
                    rotate_v=rng.random() < 0.8, fused=rng.random() < 0.5, paged=rng.random() < 0.5,
                    padding=rng.choice([0, 0, 13]))
    if kind == "calibrate":
        return dict(kind="calibrate", rows=_log(rng, 1000, 200000), constants=rng.choice([1, 3, 7, 16, 46]),
                    dtype=rng.choice(["float32", "bfloat16"]), rotate=rng.random() < 0.7, pow2=rng.random() < 0.5)
    d, cache = 128, "fp4"
    if kind == "head":
        d = rng.choice([64, 256])
    if kind == "ref":
        cache = rng.choice(["fp8", "bf16", "tq4"])
    hkv = rng.choice([1, 2, 3, 4, 8])
    g = rng.choice([1, 4, 5, 6, 8, 8, 12, 16])
    b = _log(rng, 1, 128)
    per_token = hkv * (REF_BYTES[cache] if cache in REF_BYTES else 17 * d // 16)
    ctx = _log(rng, 16, min(131072, max(64, 1.5e9 / (b * per_token))))
    spread = rng.choice([0.0, 0.3, 0.8])
    high = min(131072, 8 * ctx)
    prefix = 0
    if kind == "cascade":
        ctx = max(ctx, 512)
        high = max(high, 1024)
        prefix = PAGE * max(1, int(ctx * rng.uniform(0.1, 0.9)) // PAGE)
    bound = 0 if rng.random() < 0.6 else max(1024, 1 << (high - 1).bit_length())
    case = _decode("", "attention" if kind == "attention" else "cascade" if kind == "cascade" else "step", cache=cache,
                   batch=b, q_heads=hkv * g, kv_heads=hkv, head_dim=d, context=ctx, spread=spread, low=1, high=high,
                   lens=rng.randrange(1 << 16), bound=bound, partition=rng.choice([0, 0, 0, 0, 512, 4096]),
                   dtype=rng.choice(["bfloat16", "bfloat16", "float16", "float32"]),
                   out=rng.choice(["bfloat16", "float32"]), rotate_v=rng.random() < 0.7,
                   fp8_query=kind == "attention" and rng.random() < 0.5, prefix=prefix)
    del case["name"]
    return case


def lengths(case):
    """The batch's context lengths, a function of the case alone."""
    r = random.Random(case["lens"])
    if not case["spread"]:
        return [case["context"]] * case["batch"]
    return [min(max(int(case["context"] * math.exp(case["spread"] * r.gauss(0, 1))), case["low"]), case["high"])
            for _ in range(case["batch"])]


class _Plan:
    """Lengths in this seed's order, page table, slots of every stored token.
    Stored tokens: the shared prefix (cascade), then each sequence's own
    tokens from position own_from[b] on."""

    def __init__(self, case, seed):
        rng = np.random.default_rng(seed)
        n = np.array(lengths(case), dtype=np.int64)[rng.permutation(case["batch"])]
        s = case["prefix"]
        # whole pages of the prefix, before the sequence's last token (a shorter sequence owns its last page)
        self.own_from = np.minimum(s, (n - 1) // PAGE * PAGE) if s else np.zeros_like(n)
        own_pages = (n - self.own_from + PAGE - 1) // PAGE
        num_pages = int(s // PAGE + own_pages.sum()) + 3
        perm = rng.permutation(num_pages)
        self.max_context = max(case["bound"], int(n.max()))
        width = -(-self.max_context // PAGE)
        table = np.zeros((case["batch"], width), dtype=np.int32)
        self.prefix_pages = perm[:s // PAGE]
        cur = s // PAGE
        slots = [self.prefix_pages[np.arange(s) // PAGE] * PAGE + np.arange(s) % PAGE]
        for b in range(case["batch"]):
            lo, shared = int(self.own_from[b]), int(self.own_from[b]) // PAGE
            table[b, :shared] = self.prefix_pages[:shared]
            table[b, shared:shared + own_pages[b]] = perm[cur:cur + own_pages[b]]
            cur += int(own_pages[b])
            pos = np.arange(lo, int(n[b]))
            slots.append(table[b, pos // PAGE].astype(np.int64) * PAGE + pos % PAGE)
        self.lens, self.num_pages, self.table = n, num_pages, table
        self.slots = np.concatenate(slots)
        self.first = s + np.concatenate([[0], np.cumsum(n - self.own_from)])   # stored index of a sequence's own tokens


def _gains(rng, kv_heads, d):
    """[Hkv, d]: 20 at 4 outlier channels per head."""
    g = np.ones((kv_heads, d), dtype=np.float32)
    for h in range(kv_heads):
        g[h, rng.permutation(d)[:4]] = 20.0
    return torch.as_tensor(g, device="cuda")


def _tokens(case, seed, count):
    """(lo, hi, K, V) of the stored tokens, in chunks of about 64M elements."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    rng = np.random.default_rng(seed + 1)
    h, d, dt = case["kv_heads"], case["head_dim"], DTYPES[case["dtype"]]
    gk, gv = _gains(rng, h, d).to(dt), _gains(rng, h, d).to(dt)
    step = max(PAGE, (1 << 26) // (h * d))
    for lo in range(0, count, step):
        hi = min(count, lo + step)
        k = torch.randn((hi - lo, h, d), generator=gen, device="cuda", dtype=dt)
        v = torch.randn((hi - lo, h, d), generator=gen, device="cuda", dtype=dt)
        yield lo, hi, k.mul_(gk), v.mul_(gv)


def _query(case, seed):
    """The queries and the step's new K and V rows."""
    gen = torch.Generator(device="cuda").manual_seed(seed + 7)
    b, d, dt = case["batch"], case["head_dim"], DTYPES[case["dtype"]]
    rows = [torch.randn((b, n, d), generator=gen, device="cuda", dtype=dt)
            for n in (case["q_heads"], case["kv_heads"], case["kv_heads"])]
    return rows


def _desc(case, num_pages):
    if case["cache"] == "fp4":
        return uq.CacheDesc(num_kv_heads=case["kv_heads"], num_pages=num_pages, c=C, rotate_v=case["rotate_v"],
                            head_dim=case["head_dim"])
    return uq.RefCacheDesc(num_kv_heads=case["kv_heads"], num_pages=num_pages, fmt=case["cache"], k_scale=REF_SCALE,
                           v_scale=REF_SCALE, codebook=np.array(CODEBOOK, np.float32) if case["cache"] == "tq4" else None)


def _write_inputs(case, seed):
    """K and V rows (views of one fused QKV buffer when `fused`), slots and,
    when `paged`, the page table of 8 sequences the logical slots go through."""
    rng = np.random.default_rng(seed)
    t, h, d = case["tokens"], case["kv_heads"], case["head_dim"]
    rows = torch.cat([torch.cat([k, v], 1) for _, _, k, v in _tokens(case, seed, t)])
    if case["fused"]:   # 4 query heads' channels in front of K and V
        buf = torch.zeros((t, 4 + 2 * h, d), dtype=rows.dtype, device="cuda")
        buf[:, 4:] = rows
        k, v = buf[:, 4:4 + h], buf[:, 4 + h:]
    else:
        k, v = rows[:, :h].contiguous(), rows[:, h:].contiguous()
    per_seq = -(-t // 8)   # 8 sequences' tokens one after another
    width = -(-per_seq // PAGE)
    num_pages = 8 * width + 5
    table = rng.permutation(num_pages)[:8 * width].reshape(8, width).astype(np.int32)
    seq, pos = np.arange(t) // per_seq, np.arange(t) % per_seq
    slots = seq * (width * PAGE) + pos if case["paged"] else table[seq, pos // PAGE].astype(np.int64) * PAGE + pos % PAGE
    slots = slots.astype(np.int64)
    if case["padding"]:
        slots[rng.permutation(t)[:min(case["padding"], t // 2)]] = -1
    return k, v, torch.as_tensor(slots, device="cuda"), torch.as_tensor(table, device="cuda"), num_pages


def _calibrate_inputs(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    gain = _gains(np.random.default_rng(seed), 1, 128)
    x = torch.randn((case["rows"], 128), generator=gen, device="cuda").mul_(gain).to(DTYPES[case["dtype"]])
    return x, torch.linspace(0.05, 0.5, case["constants"], device="cuda")


def prepare(case, seed):
    if case["kind"] == "calibrate":
        x, c = _calibrate_inputs(case, seed)
        return dict(case=case, x=x, c=c)
    if case["kind"] == "write":
        k, v, slots, table, num_pages = _write_inputs(case, seed)
        desc = _desc(case, num_pages)
        pools = desc.alloc_pools(fill=0) if case["cache"] == "fp4" else (desc.alloc_cache(fill=0),)
        return dict(case=case, desc=desc, k=k, v=v, slots=slots, table=table if case["paged"] else None, pools=pools)
    plan = _Plan(case, seed)
    desc = _desc(case, plan.num_pages)
    pools = desc.alloc_pools(fill=0) if case["cache"] == "fp4" else (desc.alloc_cache(fill=0),)
    slots = torch.as_tensor(plan.slots, device="cuda")
    write = uq.quantize_kv if case["cache"] == "fp4" else uq.ref_write_kv
    for lo, hi, k, v in _tokens(case, seed, len(plan.slots)):
        write(desc, k, v, slots[lo:hi], *pools)
    q, k_new, v_new = _query(case, seed)
    b, hq = case["batch"], case["q_heads"]
    table = torch.as_tensor(plan.table, device="cuda")
    lens = torch.as_tensor(plan.lens.astype(np.int32), device="cuda")
    state = dict(case=case, desc=desc, pools=pools, q=q, k_new=k_new, v_new=v_new, table=table, lens=lens,
                 max_context=plan.max_context, scale=case["head_dim"] ** -0.5,
                 out=torch.empty((b, hq, case["head_dim"]), dtype=DTYPES[case["out"]], device="cuda"))
    if case["kind"] == "cascade":
        state["prefix"] = uq.SharedPrefix(torch.as_tensor(plan.prefix_pages.astype(np.int32), device="cuda"),
                                          torch.as_tensor(plan.own_from.astype(np.int32), device="cuda"),
                                          case["prefix"])
        n = uq.cascade_workspace_bytes(case["kv_heads"], b, hq, plan.max_context, state["prefix"], case["partition"])
        state["workspace"] = torch.empty(n, dtype=torch.uint8, device="cuda")
    elif case["cache"] == "fp4":
        state["workspace"] = uq.alloc_workspace(desc, b, hq, plan.max_context, case["partition"])
    else:
        state["workspace"] = uq.ref_alloc_workspace(desc, b, hq, plan.max_context, case["partition"])
    if case["fp8_query"]:
        state["q8"] = torch.empty(q.shape, dtype=torch.uint8, device="cuda")
    if case["kind"] == "step" and case["head_dim"] != 128:
        # the append's logical slots: every sequence's last position
        state["append"] = (torch.arange(b, device="cuda") * (table.shape[1] * PAGE) + lens.long() - 1)
    return state


def run(s):
    case = s["case"]
    if case["kind"] == "calibrate":
        return uq.quantize_error(s["x"], s["c"], case["rotate"], case["pow2"])
    if case["kind"] == "write":
        if case["cache"] == "fp4":
            uq.quantize_kv(s["desc"], s["k"], s["v"], s["slots"], *s["pools"], page_table=s["table"])
        else:
            uq.ref_write_kv(s["desc"], s["k"], s["v"], s["slots"], *s["pools"], page_table=s["table"])
        return list(s["pools"])
    rest = (s["table"], s["lens"], s["max_context"])
    kw = dict(softmax_scale=s["scale"], partition_tokens=case["partition"], workspace=s["workspace"], out=s["out"])
    if case["kind"] == "attention":
        q = s["q"]
        if case["fp8_query"]:
            q = uq.prepare_query(s["desc"], q, out=s["q8"])
        return [uq.decode_attention(s["desc"], q, *s["pools"], *rest, **kw)]
    if case["kind"] == "cascade":
        uq.decode_cascade(s["desc"], s["q"], *s["pools"], *rest, s["prefix"], k_new=s["k_new"], v_new=s["v_new"], **kw)
    elif case["cache"] != "fp4":
        uq.ref_decode_step(s["desc"], s["q"], s["k_new"], s["v_new"], *s["pools"], *rest, **kw)
    elif case["head_dim"] == 128:
        uq.decode_step(s["desc"], s["q"], s["k_new"], s["v_new"], *s["pools"], *rest, **kw)
    else:
        uq.quantize_kv(s["desc"], s["k_new"], s["v_new"], s["append"], *s["pools"], page_table=s["table"])
        uq.decode_attention(s["desc"], s["q"], *s["pools"], *rest, **kw)
    return [s["out"], *s["pools"]]


def _token_heads(case):
    """(tokens x KV heads of distinct stored context, tokens x query heads attended)."""
    n = lengths(case)
    stored = sum(n)
    if case["kind"] == "cascade":
        shared = [min(case["prefix"], (x - 1) // PAGE * PAGE) for x in n]
        stored += max(shared) - sum(shared)
    return stored * case["kv_heads"], sum(n) * case["q_heads"]


def work(case):
    if case["kind"] == "calibrate":
        item = 4 if case["dtype"] == "float32" else 2
        # the rotation's 7 adds per value, then per constant: encode, decode, subtract, square and add
        return {"bytes": case["rows"] * 128 * item, "flops": case["rows"] * 128 * (7 + 5 * case["constants"])}
    d, item = case["head_dim"], 4 if case["dtype"] == "float32" else 2
    per = REF_BYTES[case["cache"]] if case["cache"] in REF_BYTES else 17 * d // 16
    if case["kind"] == "write":
        n = case["tokens"] * case["kv_heads"]
        return {"bytes": n * (2 * d * item + per) + 8 * case["tokens"], "flops": n * 2 * d * (int(math.log2(d)) + 3)}
    stored, attended = _token_heads(case)
    rows = case["batch"] * case["q_heads"] * d
    new = 0 if case["kind"] == "attention" else case["batch"] * case["kv_heads"] * (2 * d * item + per)
    return {"bytes": stored * per + rows * (item + (2 if case["out"] == "bfloat16" else 4)) + new,
            "flops": 4 * attended * d}


def tolerance(case):
    if case["kind"] == "write":
        return "exact"
    if case["kind"] == "calibrate":
        return {"rel": 1e-6, "max": 1e-5}
    if case["out"] == "bfloat16":
        return {"rel": 4e-3, "max": 2e-2}   # half a unit of bf16's last place is 2e-3
    if case["cache"] == "fp8":
        return {"rel": 2e-3, "max": 5e-2}   # the FP8 x FP8 matrix instruction alone is 3e-4 off 64 bits
    return {"rel": 3e-5, "max": 2e-3}       # 1.4e-6 to 8.1e-6 off 64 bits measured over contexts of 16 to 32768 tokens


# --------------------------------------------------------------------------
# The same results from plain torch in 64 bits.  What the formats store is
# decided in fp32 (the rotation's butterfly, c times the group maximum), so
# the encoders below follow those fp32 values; everything after is 64 bits.


def _wht(x):
    """Walsh-Hadamard transform of the last dimension: stages 1, 2, 4, ...,
    (a, b) -> (a + b, a - b), then one multiply by 1/sqrt(d) in x's type."""
    d, shape = x.shape[-1], x.shape
    h = 1
    while h < d:
        y = x.reshape(*shape[:-1], d // (2 * h), 2, h)
        a, b = y[..., 0, :], y[..., 1, :]
        x = torch.stack([a + b, a - b], dim=-2).reshape(shape)
        h *= 2
    return x * torch.tensor(1 / math.sqrt(d), dtype=x.dtype, device=x.device)


def _e2m1(y):
    """Nearest of 0, .5, 1, 1.5, 2, 3, 4, 6 (ties to the even code), signed."""
    m = y.abs()
    idx = ((m > 0.25).int() + (m >= 0.75) + (m > 1.25) + (m >= 1.75) + (m > 2.5) + (m >= 3.5) + (m > 5.0))
    lv = torch.tensor([0.0, 0.5, 1.0, 1.5, 2.0, 3.0, 4.0, 6.0], device=y.device)
    return torch.copysign(lv[idx.long()], y)


def _pow2_scale(m, c):
    """2^round(log2(c m)) of the cache format, from the fp32 bits of c m (c m normal)."""
    y = m * c
    e = (((y.view(torch.int32) + 0x4AFB0C) >> 23).clamp(max=254) - 127).float()
    return torch.where(y > 0, torch.exp2(e), torch.zeros_like(y))


def _fp4(x, rotate):
    """fp32 rows -> the values their FP4 codes and scales stand for."""
    if rotate:
        x = _wht(x)
    g = x.reshape(*x.shape[:-1], -1, 32)
    s = _pow2_scale(g.abs().amax(-1, keepdim=True), torch.tensor(C, dtype=torch.float32, device=x.device))
    return (_e2m1(g / torch.where(s > 0, s, torch.ones_like(s))) * s).reshape(x.shape)


def _e4m3(x):
    return x.clamp(-448, 448).to(torch.float8_e4m3fn).float()


def _store(case, k, v):
    """(K values, K row factors or None, V values) of what the cache stores, all exact in bf16 or fp32."""
    k, v = k.float(), v.float()
    if case["cache"] == "fp4":
        return _fp4(k, True).bfloat16(), None, _fp4(v, case["rotate_v"]).bfloat16()
    if case["cache"] == "fp8":
        return _e4m3(k / REF_SCALE).bfloat16(), None, _e4m3(v / REF_SCALE).bfloat16()
    if case["cache"] == "bf16":
        return k.bfloat16(), None, v.bfloat16()
    lv = torch.tensor(CODEBOOK, dtype=torch.float32, device=k.device).bfloat16().double()
    mid = (lv[1:] + lv[:-1]) / 2
    k = _wht(k).double()
    n = k.square().sum(-1).sqrt().float()
    idx = torch.zeros_like(k, dtype=torch.int8)
    for j in range(15):
        idx += (k > mid[j] * n.double()[..., None])
    k = lv.bfloat16()[idx.long()]
    g = v.reshape(*v.shape[:-1], -1, 32)
    z = g.amin(-1, keepdim=True).bfloat16().float()
    # (a tensor divisor: torch multiplies by the reciprocal of a scalar one on the GPU)
    s = ((g.amax(-1, keepdim=True) - z).clamp(min=0) / torch.full_like(z, 15.0)).bfloat16().float()
    code = torch.where(s > 0, ((g - z) / torch.where(s > 0, s, torch.ones_like(s))).round().clamp(0, 15),
                       torch.zeros_like(g))
    return k, n, (s.double() * code + z).float().bfloat16().reshape(v.shape)


def _exact_query(case, q):
    q = q.float()
    if case["cache"] == "fp4":
        return _e4m3(_wht(q)).double()
    if case["cache"] == "fp8":
        return _e4m3(q).double()
    return (_wht(q) if case["cache"] == "tq4" else q).bfloat16().double()


def _exact_calibrate(case, seed):
    x, cs = _calibrate_inputs(case, seed)
    sums = torch.zeros((case["constants"], 2), dtype=torch.float64, device="cuda")
    for lo in range(0, case["rows"], 1 << 16):
        g = x[lo:lo + (1 << 16)].float()
        g = (_wht(g) if case["rotate"] else g).reshape(-1, 4, 32)
        m = g.abs().amax(-1, keepdim=True)
        sums[:, 1] += g.double().square().sum()
        for i in range(case["constants"]):
            s = _pow2_scale(m, cs[i]) if case["pow2"] else m * cs[i]
            y = _e2m1(g / torch.where(s > 0, s, torch.ones_like(s)))
            sums[i, 0] += (g.double() - y.double() * s.double()).square().sum()
    return sums


def exact(case, seed):
    if case["kind"] == "write" or case["kind"] != "calibrate" and sum(lengths(case)) * case["kv_heads"] > 3e7:
        return None   # bytes; or over 20 seconds in 64 bits
    if case["kind"] == "calibrate":
        return _exact_calibrate(case, seed)
    plan = _Plan(case, seed)
    stored = [_store(case, k, v) for _, _, k, v in _tokens(case, seed, len(plan.slots))]
    k_all, v_all = torch.cat([s[0] for s in stored]), torch.cat([s[2] for s in stored])
    n_all = torch.cat([s[1] for s in stored]) if stored[0][1] is not None else None
    q, k_new, v_new = _query(case, seed)
    if case["kind"] != "attention":   # the step's token is the last one of its sequence
        last = torch.as_tensor(plan.first[1:] - 1, device="cuda")
        kn, nn, vn = _store(case, k_new, v_new)
        k_all[last], v_all[last] = kn, vn
        if nn is not None:
            n_all[last] = nn
    q = _exact_query(case, q)
    d, hkv = case["head_dim"], case["kv_heads"]
    scale = float(np.float32(d ** -0.5)) * (REF_SCALE if case["cache"] == "fp8" else 1.0)
    out = torch.empty((case["batch"], case["q_heads"], d), dtype=torch.float64, device="cuda")
    for b in range(case["batch"]):
        rows = torch.cat([torch.arange(int(plan.own_from[b])),
                          torch.arange(int(plan.first[b]), int(plan.first[b + 1]))]).to("cuda")
        kb = k_all[rows].double().permute(1, 2, 0).contiguous()          # [Hkv, d, n]
        sc = torch.bmm(q[b].reshape(hkv, -1, d), kb) * scale             # [Hkv, G, n]
        del kb
        if n_all is not None:
            sc = sc * n_all[rows].double().t()[:, None, :]
        vb = v_all[rows].double().permute(1, 0, 2).contiguous()          # [Hkv, n, d]
        out[b] = torch.bmm(torch.softmax(sc, -1), vb).reshape(-1, d)
    if case["cache"] == "fp8":
        out = out * REF_SCALE
    if case["cache"] == "fp4" and case["rotate_v"]:
        out = _wht(out)
    return [out] if case["kind"] == "attention" else [out] + [None] * (2 if case["cache"] == "fp4" else 1)
