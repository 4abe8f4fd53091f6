"""uq_quantize_error at the edges of its units: 1 row to beyond one pass of the
grid (16 rows per wave, 16 waves per block, 512 blocks), 1 to 5 constants (two
at a time, then one) and 256, both scale rules, accumulation into given sums.
Oracle: the same sums in fp64 for small sets; the large set against the sum
over its halves.  The kernel sums squares in fp32 over a lane's 32 values and
the wave's 64 lanes (38 roundings of positive terms, 38 * 2^-24 = 2.3e-6) and in
fp64 from there, and each square carries 2 more roundings: held to 4e-6."""
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


@pytest.mark.parametrize("rows,constants,pow2", [(1, 1, True), (15, 2, False), (16, 3, True), (17, 5, False),
                                                 (65, 4, True), (257, 2, True), (1000, 256, True)])
def test_small_sets(uq, rows, constants, pow2):
    dev = torch.device("cuda:0")
    print(f"quantize_error: {rows} rows, {constants} constants, pow2 {pow2}", flush=True)
    x = np.random.default_rng(rows).standard_normal((rows, 128)).astype(np.float32)
    x[0, 32:64] = 0.0   # an all-zero group when the rows are not rotated
    c = np.linspace(0.05, 0.5, constants, dtype=np.float32)
    for rotate in (True, False):
        got = uq.quantize_error(torch.as_tensor(x, device=dev), torch.as_tensor(c, device=dev), rotate, pow2)
        ref = oracle.quantize_error(x, c, rotate, pow2)
        torch.cuda.synchronize()
        assert np.allclose(got.cpu().numpy(), ref, rtol=4e-6, atol=0)


def test_more_rows_than_one_pass_of_the_grid(uq):
    dev = torch.device("cuda:0")
    rows = 16 * 16 * 512 + 16 * 512 + 5
    print(f"quantize_error: {rows} rows", flush=True)
    x = torch.randn((rows, 128), generator=torch.Generator(device=dev).manual_seed(1), device=dev)
    c = torch.tensor([0.156, 0.195, 1.0], device=dev)
    whole = uq.quantize_error(x, c)
    halves = uq.quantize_error(x[:rows // 2], c)
    uq.quantize_error(x[rows // 2:], c, sums=halves)
    torch.cuda.synchronize()
    assert torch.allclose(whole, halves, rtol=4e-6, atol=0)
