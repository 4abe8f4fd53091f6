"""The merge of balanced splits in which a few long contexts among many short
ones take far more partials than the average row (over 16: merged by a block
per row, ahead of the launch's other blocks).

  * results against the same call with an explicit partition.  The two paths
    round every softmax weight to two BF16 terms, |error| <= 2^-16 of it, so the
    errors of a row are 2^-16 of terms whose sum is the row: over zero-mean V the
    errors and the row itself grow alike, and a (sequence, head) row differs by
    about 2^-16 = 1.5e-5 relative L2.  Held to 1e-4; a token of n lost or counted
    twice moves a row by about 1 / sqrt(n), 2.9e-3 or more here;
  * the merge launch alone takes at most twice as long for one long context
    among 31 short ones as for 32 equal ones (16 lanes that walk the long rows
    one partial after another: 2.2 times as long, from a warm cache).
"""
import numpy as np
import pytest
import torch

from paper_2606_20474_amd import workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def uq():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2606_20474_amd import uq as mod
    return mod


def lengths(batch, longs, top):
    """`longs` contexts near `top` at both ends and spread over the batch, the others short or empty."""
    rng = np.random.default_rng(batch)
    ctx = rng.integers(0, 300, batch)
    ctx[np.linspace(0, batch - 1, longs).astype(int)] = top - 77 * np.arange(longs)
    return [int(c) for c in ctx]


@pytest.mark.parametrize("batch,hq,hkv,longs,top,d,fmt", [
    (16, 64, 8, 1, 60001, 128, "fp4"),     # 4 rows on average: 16 lanes per row
    (8, 16, 8, 1, 60001, 128, "fp4"),      # 8 rows on average: a wave per row
    (64, 64, 8, 5, 20000, 128, "fp4"),     # more long rows than blocks for them; one length per planner lane
    (65, 64, 8, 5, 20000, 128, "fp4"),     # two lengths per planner lane
    (256, 24, 8, 3, 40000, 128, "fp4"),    # four
    (200, 5, 1, 2, 30000, 128, "fp4"),
    (100, 4, 2, 3, 20000, 256, "fp4"),
    (90, 8, 1, 2, 40000, 64, "fp4"),
    (90, 16, 2, 2, 40000, 64, "fp4"),
    (70, 16, 8, 3, 12000, 128, "bf16"),
])
def test_long_rows(uq, batch, hq, hkv, longs, top, d, fmt):
    dev = torch.device("cuda:0")
    print(f"long rows: B={batch} {hq}/{hkv} heads of {d}, {longs} of {top}, {fmt}", flush=True)
    wl = workloads.custom(batch, hq, hkv, lengths(batch, longs, top), seed=batch, head_dim=d)
    if fmt == "fp4":
        desc = uq.CacheDesc(num_kv_heads=hkv, num_pages=wl.num_pages, head_dim=d)
        bufs, write, attend, nbytes = desc.alloc_pools(dev, fill=0), uq.quantize_kv, uq.decode_attention, uq.workspace_bytes
    else:
        desc = uq.RefCacheDesc(num_kv_heads=hkv, num_pages=wl.num_pages, fmt=fmt)
        bufs, write, attend, nbytes = (desc.alloc_cache(dev, fill=0),), uq.ref_write_kv, uq.ref_decode_attention, uq.ref_workspace_bytes
    for key, lo, hi, row in wl.segments():
        k, v = wl.kv(key, lo, hi, device=dev)
        write(desc, k, v, torch.as_tensor(wl.slots(key, lo, hi, row), device=dev), *bufs)
    q, pt = wl.q.to(dev), torch.as_tensor(wl.page_table, device=dev)
    ctx = torch.as_tensor(wl.context_lens, device=dev)
    ws = torch.full((nbytes(desc, batch, hq, wl.max_context, 0),), 0xFF, dtype=torch.uint8, device=dev)
    got = attend(desc, q, *bufs, pt, ctx, wl.max_context, d ** -0.5, 0, workspace=ws).double()
    ref = attend(desc, q, *bufs, pt, ctx, wl.max_context, d ** -0.5, 1536).double()   # not a default partition
    rel = (got - ref).norm(dim=-1) / ref.norm(dim=-1).clamp(min=1e-30)
    print(f"  largest relative L2 of a row {float(rel.max()):.2e}", flush=True)
    assert torch.all(got[ctx == 0] == 0)
    assert float(rel[ctx > 0].max()) <= 1e-4


def test_merge_time_of_a_skewed_batch(uq):
    dev = torch.device("cuda:0")
    batch, hq, hkv, bound = 32, 64, 8, 120000
    desc = uq.CacheDesc(num_kv_heads=hkv, num_pages=1)
    ws = uq.alloc_workspace(desc, batch, hq, bound, 0, dev).zero_()   # weights 0: the times do not depend on the values
    out = torch.empty((batch, hq, 128), device=dev)
    start, stop = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)

    def time(ctx):
        ctx = torch.tensor(ctx, dtype=torch.int32, device=dev)
        times = []
        for _ in range(7):
            torch.cuda.synchronize()
            start.record()
            for _ in range(50):
                uq.decode_merge(desc, batch, hq, ctx, bound, 0, ws, out)
            stop.record()
            torch.cuda.synchronize()
            times.append(start.elapsed_time(stop) * 20)
        return min(times)

    equal, skewed = time([4700] * batch), time([bound] + [1000] * (batch - 1))
    print(f"merge: equal {equal:.1f} us, skewed {skewed:.1f} us", flush=True)
    assert skewed <= 2 * equal


@pytest.mark.parametrize("hq,hkv", [(8, 8), (32, 8), (40, 8), (64, 8), (96, 8), (128, 8), (64, 16), (36, 9)])
@pytest.mark.parametrize("partition", [1536, 512, 64])   # up to 3, 8 and 63 partials: 16 lanes, a wave, a block per row
def test_query_heads_of_fixed_partitions(uq, hq, hkv, partition):
    """Every group size and merge form writes every query head (KV heads a
    multiple of 8: the heads of a block belong to one KV head), against one
    partition per sequence, finished without a merge."""
    dev = torch.device("cuda:0")
    print(f"merge of fixed partitions: {hq}/{hkv} heads, partition {partition}", flush=True)
    wl = workloads.custom(4, hq, hkv, [4000, 1537, 65, 3100], seed=hq, head_dim=128)
    desc = uq.CacheDesc(num_kv_heads=hkv, num_pages=wl.num_pages)
    pools = desc.alloc_pools(dev, fill=0)
    for key, lo, hi, row in wl.segments():
        k, v = wl.kv(key, lo, hi, device=dev)
        uq.quantize_kv(desc, k, v, torch.as_tensor(wl.slots(key, lo, hi, row), device=dev), *pools)
    q, pt = wl.q.to(dev), torch.as_tensor(wl.page_table, device=dev)
    ctx = torch.as_tensor(wl.context_lens, device=dev)
    out = [uq.decode_attention(desc, q, *pools, pt, ctx, wl.max_context, 128 ** -0.5, p,
                               out=torch.full((4, hq, 128), float("nan"), device=dev)).double() for p in (partition, 4000)]
    assert torch.isfinite(out[0]).all()
    assert float(((out[0] - out[1]).norm(dim=-1) / out[1].norm(dim=-1)).max()) <= 1e-4
