"""Balanced splits of batches whose lengths are (nearly) equal: every context is
cut into the same number of parts, chosen so that no CU gets a block more than it
need.

  * results against the same call with an explicit partition; both round every
    softmax weight to two BF16 terms, |error| <= 2^-16 of it, so over zero-mean V
    a (sequence, head) row differs by about 2^-16 relative L2: held to 1e-4 (a token
    of n lost or counted twice moves a row by about 1 / sqrt(n), 1.5e-2 or more
    here).  One, two, three parts and parts that end on an odd page; lengths at the
    edges of the 128-token unit; lengths on both sides of the rule's threshold (15/16
    of the longest on average), with an empty one; bounds above the lengths; one and
    up to four lengths per planner lane; every format and head size;
  * 36 contexts of 100k, 4 KV heads: the default call takes at most 1.07 times
    as long as an explicit cut into three (the most parts that fit, four: 1.15).
"""
import pytest
import torch

from paper_2606_20474_amd import workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def uq():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2606_20474_amd import uq as mod
    return mod


def same(n):
    return lambda b: [n] * b


def near(n, step, empty=False):
    """n and shorter, `step` apart in a cycle of 16."""
    return lambda b: [0 if empty and i == b // 2 else n - step * (i * 7 % 16) for i in range(b)]


@pytest.mark.parametrize("batch,hq,hkv,lens,bound,fmt,d", [
    (100, 8, 4, same(1300), 0, "fp4", 128),             # one part each, finished in place
    (100, 8, 4, same(1300), 4000, "fp4", 128),          # the same under a bound that allows more
    (48, 16, 8, same(2900), 0, "fp4", 128),             # two
    (48, 16, 8, same(2816), 0, "fp4", 128),             # two of exactly 11 units
    (48, 16, 8, same(2817), 0, "fp4", 128),             # one token more
    (36, 8, 4, same(4001), 0, "fp4", 128),              # three
    (36, 8, 4, near(4001, 30), 0, "fp4", 128),          # 225 of 4001 below it on average: inside 1/16
    (36, 8, 4, near(4001, 40), 0, "fp4", 128),          # 300: outside
    (36, 8, 4, near(4001, 20, True), 0, "fp4", 128),    # an empty one
    (130, 8, 8, near(2100, 8), 4096, "fp4", 128),       # up to four lengths per planner lane
    (256, 8, 4, same(1100), 0, "fp4", 128),
    (48, 16, 8, same(2900), 0, "fp8", 128),
    (48, 16, 8, near(2900, 11), 0, "bf16", 128),
    (48, 16, 8, same(2900), 0, "tq4", 128),
    (72, 32, 8, same(2900), 0, "fp4", 64),              # two KV heads per block
    (200, 5, 5, near(1500, 5), 0, "fp4", 64),           # two page pairs of one KV head
    (100, 48, 4, same(1300), 0, "fp4", 64),
    (48, 16, 8, same(2900), 0, "fp4", 256),
])
def test_equal_lengths(uq, batch, hq, hkv, lens, bound, fmt, d):
    dev = torch.device("cuda:0")
    ctx = lens(batch)
    print(f"equal split: B={batch} {hq}/{hkv} heads of {d}, up to {max(ctx)}, bound {bound}, {fmt}", flush=True)
    wl = workloads.custom(batch, hq, hkv, ctx, seed=batch, head_dim=d)
    top = max(bound, wl.max_context)
    if fmt == "fp4":
        desc = uq.CacheDesc(num_kv_heads=hkv, num_pages=wl.num_pages, head_dim=d)
        bufs, write, attend, nbytes = desc.alloc_pools(dev, fill=0), uq.quantize_kv, uq.decode_attention, uq.workspace_bytes
        partials, merge = uq.decode_partials, uq.decode_merge
    else:
        desc = uq.RefCacheDesc(num_kv_heads=hkv, num_pages=wl.num_pages, fmt=fmt)
        bufs, write, attend, nbytes = (desc.alloc_cache(dev, fill=0),), uq.ref_write_kv, uq.ref_decode_attention, uq.ref_workspace_bytes
        partials, merge = uq.ref_decode_partials, uq.ref_decode_merge
    for key, lo, hi, row in wl.segments():
        k, v = wl.kv(key, lo, hi, device=dev)
        write(desc, k, v, torch.as_tensor(wl.slots(key, lo, hi, row), device=dev), *bufs)
    q, n = wl.q.to(dev), torch.as_tensor(wl.context_lens, device=dev)
    pt = torch.zeros((batch, -(-top // 16)), dtype=torch.int32, device=dev)
    pt[:, :wl.page_table.shape[1]] = torch.as_tensor(wl.page_table, device=dev)
    ws = torch.full((nbytes(desc, batch, hq, top, 0),), 0xFF, dtype=torch.uint8, device=dev)
    got = attend(desc, q, *bufs, pt, n, top, d ** -0.5, 0, workspace=ws)
    ref = attend(desc, q, *bufs, pt, n, top, d ** -0.5, 592)   # whole pages, but not units
    ws.fill_(0xFF)
    two = torch.full_like(got, float("nan"))
    partials(desc, q, *bufs, pt, n, top, d ** -0.5, 0, ws, two)
    merge(desc, batch, hq, n, top, 0, ws, two)
    assert torch.equal(two, got)
    rel = (got.double() - ref.double()).norm(dim=-1) / ref.double().norm(dim=-1).clamp(min=1e-30)
    print(f"  largest relative L2 of a row {float(rel.max()):.2e}", flush=True)
    assert torch.all(got[n == 0] == 0)
    assert float(rel[n > 0].max()) <= 1e-4


def test_time_of_equal_lengths(uq):
    dev = torch.device("cuda:0")
    batch, hq, hkv, ctx = 36, 32, 4, 100000
    pages = -(-ctx // 16)
    desc = uq.CacheDesc(num_kv_heads=hkv, num_pages=batch * pages)
    codes, scales = desc.alloc_pools(dev, fill=0)
    scales.fill_(127)
    pt = torch.randperm(batch * pages, device=dev).to(torch.int32).reshape(batch, pages)
    n = torch.full((batch,), ctx, dtype=torch.int32, device=dev)
    q = torch.randn((batch, hq, 128), device=dev)
    start, stop = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    best = {}
    for _ in range(3):
        for part in (0, 33344):
            ws, out = uq.alloc_workspace(desc, batch, hq, ctx, part, dev), torch.empty((batch, hq, 128), device=dev)
            for i in range(25):
                if i == 5:
                    start.record()
                uq.decode_attention(desc, q, codes, scales, pt, n, ctx, 128 ** -0.5, part, workspace=ws, out=out)
            stop.record()
            torch.cuda.synchronize()
            best[part] = min(best.get(part, 1e9), start.elapsed_time(stop) * 50)
    print(f"36 x 100k: default {best[0]:.1f} us, cut into three {best[33344]:.1f} us", flush=True)
    assert best[0] <= 1.07 * best[33344]
