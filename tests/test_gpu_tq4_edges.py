"""Ultra-TQ key encoding where the fast decisions hand over to the exact ones:
rotated channels that are exactly zero under a codebook whose middle midpoint
is zero (ties), channels and norms at very small and very large magnitudes,
zero keys, and many random rows.  Every byte equal to the oracle's."""
import numpy as np
import pytest
import torch

import oracle
from paper_2606_20474_amd.codebook import default_tq_codebook

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def uq():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2606_20474_amd import uq as mod
    return mod


def rows():
    rng = np.random.default_rng(5)
    out = [np.zeros(128, np.float32)]
    for i, j in ((0, 64), (0, 1), (3, 77), (126, 127)):
        for s in (1.0, -1.0):
            x = np.zeros(128, np.float32)
            x[i], x[j] = 1.0, s          # half of the rotated channels cancel to zero
            out += [x, x * np.float32(1e-30), x * np.float32(3e18)]
    one = np.zeros(128, np.float32)
    one[9] = 0.37
    out += [one, np.full(128, 2.5, np.float32)]
    g = rng.standard_normal((2000, 128)).astype(np.float32)
    return np.stack(out + [r * np.float32(2.0 ** e) for r, e in zip(g, rng.integers(-60, 60, len(g)))])


@pytest.mark.parametrize("which", ["symmetric", "shifted"])
def test_bytes_match_the_oracle(uq, which):
    dev = torch.device("cuda:0")
    cb = default_tq_codebook(128)
    if which == "shifted":
        cb = (cb * np.float32(0.85) + np.float32(0.003)).astype(np.float32)
    k = rows().reshape(-1, 1, 128)
    v = np.random.default_rng(6).standard_normal(k.shape).astype(np.float32)
    pages = -(-len(k) // 16)
    slots = np.arange(len(k), dtype=np.int64)
    print(f"ultra-tq encode, {which} codebook, {len(k)} rows", flush=True)
    desc = uq.RefCacheDesc(1, pages, "tq4", codebook=cb)
    cache = desc.alloc_cache(dev, fill=0x5A)
    uq.ref_write_kv(desc, torch.as_tensor(k, device=dev), torch.as_tensor(v, device=dev),
                    torch.as_tensor(slots, device=dev), cache)
    ref = oracle.tq4_alloc_cache(pages, 1, fill=0x5A)
    oracle.tq4_write(k, v, slots, pages, cb, ref)
    torch.cuda.synchronize()
    assert np.array_equal(cache.cpu().numpy(), ref.reshape(-1))
