"""Long rows: runs that read the pair matrix, runs without one (a profiled run, a
served request) and a batch pick the same points with the same f and gains, bit
for bit, also where more candidates come near the best than are re-scored: which
of those are kept depends on the last bit of every float32 gain."""
import numpy as np
import pytest
import torch

from paper_2105_12026_amd import ebc, workloads

pytestmark = pytest.mark.gpu


def near_duplicates(n, d, seed):
    """6 points, each repeated with small noise: hundreds of gains within rounding of the best."""
    rng = np.random.default_rng([7, seed])
    x = workloads.gaussian_mixture(rng, 6, d, 6)[rng.integers(0, 6, n)]
    return (x + 1e-3 * rng.standard_normal((n, d))).astype(np.float32)


def run(t, dtype, k, full):
    ds = ebc.Dataset(t, dtype=dtype)
    ds.profile(full)
    out = [q.cpu().numpy() for q in ds.greedy(k)]
    return out, ds.sync()["window_max"]


# windows above the 256 re-scored candidates, above the 1024 listed ones, and small ones
@pytest.mark.parametrize("n,d,dtype,window", [(300, 129, "bf16", 257), (700, 200, "f16", 257), (1000, 777, "f32", 257),
                                              (2600, 300, "f32", 1025), (1500, 150, "fp8", 257), (255, 200, "bf16", 0)])
def test_with_and_without_the_pair_matrix(n, d, dtype, window):
    k = 25
    x = near_duplicates(n, d, n)
    t = torch.from_numpy(x).cuda()
    want, most = run(t, dtype, k, full=True)
    got, same = run(t, dtype, k, full=False)
    assert most >= window and same == most
    assert all(np.array_equal(a, b) for a, b in zip(got, want))
    batch = ebc.Batch([ebc.Dataset(t, dtype=dtype), ebc.Dataset(t, dtype="f32")]).greedy([k, 1])[0]
    assert all(np.array_equal(a.cpu().numpy(), b) for a, b in zip(batch, want))
    sv = ebc.Server(256 << 20, max_slots=2)
    rid = sv.submit(x, k, dtype=dtype)
    for _ in range(k + 2):
        sv.step()
    r = sv.poll(rid)
    sv.close()
    assert r["state"] == "done"
    assert all(np.array_equal(r[q], w) for q, w in zip(("sel", "f", "gain"), want))


def test_workspace_without_the_pair_matrix():
    """L1 data sets never use the matrix and take no room for it; others do without where there is none."""
    n, d = 4096, 129
    x = torch.from_numpy(near_duplicates(n, d, 1)).cuda()
    whole = ebc.lib().ebc_dataset_bytes(n, d, 0)
    matrix = 4 * n * n
    assert ebc.Dataset(x, dist="l1").workspace_bytes == whole - matrix
    ds = ebc.Dataset(x)
    assert ds.workspace_bytes == whole
    want = [q.cpu().numpy() for q in ds.greedy(9)]
    del ds
    torch.cuda.empty_cache()
    total = torch.cuda.get_device_properties(0).total_memory
    try:
        torch.cuda.set_per_process_memory_fraction((torch.cuda.memory_reserved() + matrix // 2) / total)
        ds = ebc.Dataset(x)
        got = [q.cpu().numpy() for q in ds.greedy(9)]
    finally:
        torch.cuda.set_per_process_memory_fraction(1.0)
    assert ds.workspace_bytes == whole - matrix
    assert all(np.array_equal(a, b) for a, b in zip(got, want))
