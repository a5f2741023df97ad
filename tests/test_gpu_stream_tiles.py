"""Streams in index order (each distance of a stretch made once and mirrored)
against the same stream with an order (every distance made where it lies): the
same bits, since a distance does not depend on its operands' order; and both
against the float64 oracle, f within the 1e-12 of the other stream tests. Ground
sets on both sides of the walk's register variants (256 to 4096 points and past
them), stretches that are no multiple of a 32-point tile, rows of a few values,
and few rejections per guess (the guess moves inside a group of points that is
decided together)."""
import numpy as np
import pytest
import torch

from oracle import ebc_oracle as O
from paper_2105_12026_amd import ebc
from paper_2105_12026_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dist", ["sqeuclidean", "l1"])
@pytest.mark.parametrize("n,d,k,T,batch", [
    (5, 3, 3, 1, 0), (255, 1, 6, 2, 48), (257, 17, 8, 3, 33), (513, 100, 6, 1, 64), (1025, 24, 12, 5, 100),
    (2049, 9, 5, 7, 31), (4200, 12, 6, 4, 128),
])
def test_mirrored_tiles(dist, n, d, k, T, batch):
    print(f"[gpu-case] stream tiles {dist} n={n} d={d} k={k} T={T} batch={batch}", flush=True)
    x = W.gaussian_mixture(np.random.default_rng([8, n]), n, d, min(n, 9)).astype(np.float32)
    order = torch.arange(n, dtype=torch.int32)
    ds = ebc.Dataset(torch.from_numpy(x).cuda(), dist=dist)
    three, sieve = [], []
    for o in (None, order):
        sel, f, seen = ds.three_sieves(k, 0.1, T, order=o, batch=batch)
        three.append((sel.cpu().numpy(), f.cpu().numpy(), seen))
        sel, f, v, seen = ds.sieve_streaming(k, 0.1, order=o, batch=batch)
        sieve.append((sel.cpu().numpy(), f.cpu().numpy(), v, seen))
    ds.sync()
    for a, b in (three, sieve):
        np.testing.assert_array_equal(a[0], b[0])
        np.testing.assert_array_equal(a[1], b[1])
        assert a[2:] == b[2:]
    if n > 2049:
        return
    rsel, rf, _, rseen = O.three_sieves(x, k, 0.1, T, dist=dist)
    assert three[0][0].tolist() == rsel and three[0][2] == rseen
    np.testing.assert_allclose(three[0][1], rf, rtol=1e-12)
    rsel, rf, rv, _ = O.sieve_streaming(x, k, 0.1, dist=dist)
    assert sieve[0][0].tolist() == rsel
    np.testing.assert_allclose(sieve[0][1], rf, rtol=1e-12)
