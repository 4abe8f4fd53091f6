"""Quantize-on-write at head size 256 on both sides of the line between its two
kernels (1024 units of 16 tokens of a kv head: 16 lanes per vector up to
there, 4 beyond), every pool byte against the oracle: one token, a whole unit
and one more, the last small and the first large write; zero rows (the
rotation keeps the signs of their zeros), padding, both V modes."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def uq():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2606_20474_amd import uq as mod
    return mod


@pytest.mark.parametrize("tokens,hkv,dtype,rotate_v", [
    (1, 1, torch.float32, True), (16, 3, torch.bfloat16, False), (17, 3, torch.float16, True),
    (16 * 1024, 1, torch.bfloat16, True), (16 * 1024 + 1, 1, torch.bfloat16, True), (8200, 2, torch.float32, False),
])
def test_bytes_match_the_oracle(uq, tokens, hkv, dtype, rotate_v):
    dev = torch.device("cuda:0")
    print(f"write d=256: {tokens} tokens, {hkv} kv heads, {dtype}, rotate_v {rotate_v}", flush=True)
    g = torch.Generator().manual_seed(tokens)
    k = torch.randn((tokens, hkv, 256), generator=g)
    v = torch.randn((tokens, hkv, 256), generator=g)
    k[::7] = 0.0
    v[::5] = -0.0
    k[1::11, :, 3] *= 300.0
    k, v = k.to(dtype), v.to(dtype)
    pages = -(-tokens // 16) + 2
    slots = np.random.default_rng(tokens).permutation(pages * 16)[:tokens].astype(np.int64)
    slots[3::50] = -1
    desc = uq.CacheDesc(num_kv_heads=hkv, num_pages=pages, rotate_v=rotate_v, head_dim=256)
    codes, scales = desc.alloc_pools(dev, fill=0x5A)
    uq.quantize_kv(desc, k.to(dev), v.to(dev), torch.as_tensor(slots, device=dev), codes, scales)
    pools = oracle.alloc_pools(pages, hkv, fill=0x5A, head_dim=256)
    oracle.quantize_kv(k.float().numpy(), v.float().numpy(), slots, pages, rotate_v=rotate_v, pools=pools)
    torch.cuda.synchronize()
    assert np.array_equal(codes.cpu().numpy(), pools[0])
    assert np.array_equal(scales.cpu().numpy(), pools[1])
