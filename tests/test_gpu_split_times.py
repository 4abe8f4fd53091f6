"""Times of the balanced split against fixed partitions of the default's length
(16 tokens less, so that the call does not take the split): batches of few
blocks per CU, where the order of the blocks and the length of a partition
decide which CUs finish last.  The default call may take at most 1.06 times as
long; the ratio it had, and has, stands beside each case."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def lognormal(batch, median, sigma):
    return [int(n) for n in np.random.default_rng(1).lognormal(np.log(median), sigma, batch)]


@pytest.mark.parametrize("fmt,ctx,hkv", [
    ("fp4", lognormal(80, 20000, 0.2), 4),    # 1.16, 0.95
    ("fp8", lognormal(80, 20000, 0.2), 4),    # 1.28, 0.99
    ("bf16", lognormal(80, 20000, 0.2), 4),   # 1.40, 0.96
    ("bf16", lognormal(40, 20000, 0.2), 8),   # 1.24, 0.94
    ("bf16", lognormal(20, 40000, 0.2), 8),   # 1.20, 0.96
    ("bf16", lognormal(40, 20000, 0.2), 4),   # 1.21, 0.97
    ("bf16", [30000] * 40, 8),                # 1.09, 1.00
])
def test_split_is_no_slower_than_fixed_partitions(fmt, ctx, hkv):
    from paper_2606_20474_amd import uq
    dev = torch.device("cuda:0")
    batch, hq, top = len(ctx), 8 * hkv, max(ctx)
    pages = [-(-c // 16) for c in ctx]
    order = torch.randperm(sum(pages), generator=torch.Generator().manual_seed(batch)).int()
    pt = torch.zeros((batch, -(-top // 16)), dtype=torch.int32)
    for row, ids in zip(pt, order.split(pages)):
        row[:len(ids)] = ids
    pt, n = pt.to(dev), torch.tensor(ctx, dtype=torch.int32, device=dev)
    q = torch.randn((batch, hq, 128), device=dev)
    geometry = uq.CacheDesc(num_kv_heads=hkv, num_pages=sum(pages))
    if fmt == "fp4":
        desc, attend, nbytes = geometry, uq.decode_attention, uq.workspace_bytes
        bufs = desc.alloc_pools(dev, fill=0x35)
        bufs[1].fill_(127)
    else:
        desc, attend, nbytes = uq.RefCacheDesc(num_kv_heads=hkv, num_pages=sum(pages), fmt=fmt), uq.ref_decode_attention, uq.ref_workspace_bytes
        bufs = (desc.alloc_cache(dev, fill=0x35),)
    fixed = uq.default_partition(geometry, batch, hq, top) - 16
    start, stop = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    out = torch.empty((batch, hq, 128), device=dev)
    best = {}
    for _ in range(4):
        for part in (0, fixed):
            ws = torch.empty(nbytes(desc, batch, hq, top, part), dtype=torch.uint8, device=dev)
            for i in range(20):
                if i == 5:
                    start.record()
                attend(desc, q, *bufs, pt, n, top, 128 ** -0.5, part, workspace=ws, out=out)
            stop.record()
            torch.cuda.synchronize()
            best[part] = min(best.get(part, 1e9), start.elapsed_time(stop) / 15 * 1000)
    print(f"{fmt}, {batch} contexts of {min(ctx)}-{top}, {hkv} KV heads: default {best[0]:.1f} us, partitions of {fixed} "
          f"{best[fixed]:.1f} us, {best[0] / best[fixed]:.3f}", flush=True)
    assert best[0] <= 1.06 * best[fixed]
