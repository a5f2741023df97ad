"""Sets of rows of small whole numbers, whose products and sums float32 holds
exactly, so that f is known to the rounding of its last division: groups of
sets whose member blocks fit the kept bookkeeping (12 blocks of 32 rows) to the
last, exceed it by one block, or take several rounds of it, beside short and
empty sets; rows read from the dataset's padded copy (float32, any length) and
from the caller's (a reduced-precision dataset evaluated in float32)."""
import numpy as np
import pytest
import torch

from paper_2105_12026_amd import ebc

pytestmark = pytest.mark.gpu

SIZES = {
    "kept": [250, 134, 3, 0, 256, 128, 40],   # 62 units and a set reaching out: 12 blocks
    "one over": [252, 160, 1, 255, 1, 130],   # 63 units and 40 more: 13 blocks
    "rounds": [1000, 0, 384, 385, 416, 2, 900],
}


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("sizes", list(SIZES))
@pytest.mark.parametrize("n,d", [(70, 8), (600, 33), (257, 77), (1030, 120), (513, 128)])
def test_long_sets_of_exact_rows(n, d, sizes, dtype):
    print(f"[gpu-case] long sets {sizes} {dtype} n={n} d={d}", flush=True)
    rng = np.random.default_rng([6, n, d])
    x = rng.integers(0, 4, (n, d)).astype(np.float32)
    off = np.concatenate([[0], np.cumsum(SIZES[sizes])])
    idx = rng.integers(0, n, off[-1]).astype(np.int32)
    xd = x.astype(np.float64)
    m0 = (xd * xd).sum(1)
    dist = m0[:, None] + m0[None, :] - 2.0 * (xd @ xd.T)
    ref = [np.maximum(m0 - dist[:, idx[a:b]].min(1), 0.0).sum() / n if b > a else 0.0 for a, b in zip(off, off[1:])]
    ds = ebc.Dataset(torch.from_numpy(x).cuda(), dtype=dtype)
    f = ds.eval_sets(torch.from_numpy(off), torch.from_numpy(idx)).cpu().numpy()
    ds.sync()
    np.testing.assert_allclose(f, ref, rtol=1e-15, atol=0.0)
