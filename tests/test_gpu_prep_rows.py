"""Preparation of reduced-precision rows and their grouped order: rows of small
whole numbers, which every type holds exactly, so that every product, distance
and float32 sum of the gains is exact and a gain is known to the rounding of its
division by n. Rows read four values at a time or one by one (a length that is
no multiple of 4, a pointer off 16 bytes), fewer points than a block, and more
blocks than the 256 of one round of the grouped order's counts."""
import numpy as np
import pytest
import torch

from paper_2105_12026_amd import ebc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "f16", "fp8"])
@pytest.mark.parametrize("n,d", [(1, 1), (255, 7), (513, 16), (3001, 33), (65537, 40), (70001, 33)])
def test_gains_of_exact_rows(dtype, n, d):
    print(f"[gpu-case] prep {dtype} n={n} d={d}", flush=True)
    rng = np.random.default_rng([5, n, d])
    x = rng.integers(0, 4, (n, d)).astype(np.float32)
    cand = rng.integers(0, n, 64).astype(np.int32)
    xd = x.astype(np.float64)
    m = (xd * xd).sum(1)
    dist = m[:, None] + m[cand][None, :] - 2.0 * (xd @ xd[cand].T)
    ref = np.maximum(m[:, None] - dist, 0.0).sum(0) / n
    out = []
    for shift in (0, 1):  # the second: 4 bytes off
        flat = torch.zeros(n * d + shift, device="cuda")
        flat[shift:] = torch.from_numpy(x.ravel()).cuda()
        ds = ebc.Dataset(flat[shift:].view(n, d), dtype=dtype)
        out.append(ds.marginal_gains(cand=torch.from_numpy(cand)).cpu().numpy())
        ds.sync()
    np.testing.assert_allclose(out[0], ref, rtol=4e-16, atol=0.0)
    np.testing.assert_array_equal(out[0], out[1])
