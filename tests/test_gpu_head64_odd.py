"""Head size 64 with an odd number of KV heads and at most 8 query heads each
(two page pairs of one head per iteration) against the oracle: contexts at
the edges of a page, of a page pair and of the 64-token iteration, partitions
that end on an odd page, group sizes 1, 5 and 8, both V modes; max-abs 2e-3
and relative L2 1e-3, the bars of the other head sizes' tests."""
import math

import numpy as np
import pytest
import torch

import oracle
from paper_2606_20474_amd import workloads
from test_gpu_headdim import both_caches, check, decode, uq  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu

CTX = [1, 15, 16, 17, 31, 32, 33, 48, 49, 63, 64, 65, 95, 96, 97, 127, 128, 129, 255, 257, 320, 1000, 4200, 0]


@pytest.mark.parametrize("hq,hkv", [(8, 1), (5, 1), (3, 3)])
@pytest.mark.parametrize("partition,rotate_v", [(0, True), (16, True), (48, False), (64, True), (80, True), (256, False)])
def test_decode_edges(uq, hq, hkv, partition, rotate_v):  # noqa: F811
    dev = torch.device("cuda:0")
    wl = workloads.custom(len(CTX), hq, hkv, CTX, seed=64, paging="random", rotate_v=rotate_v, head_dim=64)
    print(f"head size 64, {hq}/{hkv} heads, partition {partition}, rotate_v {rotate_v}", flush=True)
    desc, codes, scales, pools = both_caches(uq, wl, dev, fill=0xC3)
    out = decode(uq, wl, desc, codes, scales, dev, partition)
    ref = oracle.decode_attention(wl.q.numpy(), pools, wl.page_table, wl.context_lens, hkv, 1 / math.sqrt(64), rotate_v)
    assert np.all(out[-1] == 0)
    check(out, ref, f"{hq}/{hkv} p={partition}")


@pytest.mark.parametrize("hq,hkv", [(8, 1), (5, 1), (3, 3), (8, 2), (12, 1)])
@pytest.mark.parametrize("partition", [0, 16, 48, 64, 80])
def test_unwritten_tokens(uq, hq, hkv, partition):  # noqa: F811
    """Slots no token was written to hold 0xFF bytes (a scale byte of 255 is a
    NaN), the whole of physical page 0 among them, which stands in for the pages
    past the end: they do not reach the output.  Also the blocks of two KV heads
    and of one (group size above 8)."""
    dev = torch.device("cuda:0")
    wl = workloads.custom(len(CTX), hq, hkv, CTX, seed=65, paging="random", head_dim=64)
    wl.page_table = wl.page_table + 1   # page 0 belongs to no sequence
    wl.num_pages += 1
    print(f"head size 64, {hq}/{hkv} heads, partition {partition}, unwritten slots 0xFF", flush=True)
    desc, codes, scales, pools = both_caches(uq, wl, dev, fill=0xFF)
    out = decode(uq, wl, desc, codes, scales, dev, partition)
    ref = oracle.decode_attention(wl.q.numpy(), pools, wl.page_table, wl.context_lens, hkv, 1 / math.sqrt(64), True)
    assert np.all(out[-1] == 0)
    check(out, ref, f"{hq}/{hkv} p={partition}")
