"""Greedy steps that score a list of candidates (csrc/lazy.h) against steps that
score every candidate (what a profiled run does): the same picks, f and gains,
bit for bit, since both re-score the same window in float64, and against the
float64 oracle."""
import numpy as np
import pytest
import torch

from paper_2105_12026_amd import ebc, workloads

pytestmark = pytest.mark.gpu


def points(data, n, d, seed):
    rng = np.random.default_rng([91, seed])
    if data == "curves":
        return workloads.process_curves(rng, n, d).astype(np.float32)
    if data == "normal":
        return rng.standard_normal((n, d)).astype(np.float32)
    x = workloads.gaussian_mixture(rng, n, d, 12)
    if data == "outliers":
        x[: n // 50] = rng.uniform(-20.0, 20.0, (n // 50, d))
        x = x[rng.permutation(n)]
    if data == "few":  # 7 distinct points: after 7 picks every gain is 0
        x = x[rng.integers(0, 7, n)]
    if data == "sorted":  # whole stretches of one cluster
        x = x[np.argsort(x[:, 0])]
    return x.astype(np.float32)


def both(x, k, dtype, dist="sqeuclidean", graph=False):
    """(sel, f, gain, window_max) of a full-scoring run and of a default run."""
    t = torch.from_numpy(x).cuda()
    out = []
    for full in (True, False):
        ds = ebc.Dataset(t, dtype=dtype, dist=dist)
        if full:
            ds.profile(True)
        else:
            ds.set_graph(graph)
        for _ in range(2 if graph else 1):
            sel, f, gain = ds.greedy(k)
        st = ds.sync()
        out.append((sel.cpu().numpy(), f.cpu().numpy(), gain.cpu().numpy(), st["window_max"]))
    return out


# sizes: smallest that keeps lists (2048 rows), one past a block, a padded tail, many stretches; d at both ends
CASES = [
    ("mixture", 2048, 16, 30, "f32", "sqeuclidean"),
    ("mixture", 2049, 3, 30, "f32", "sqeuclidean"),
    ("outliers", 9001, 100, 40, "f32", "sqeuclidean"),
    ("sorted", 33000, 33, 25, "f32", "sqeuclidean"),
    ("normal", 5000, 128, 12, "f32", "sqeuclidean"),
    ("few", 3000, 20, 12, "f32", "sqeuclidean"),
    ("curves", 7003, 64, 30, "bf16", "sqeuclidean"),
    ("outliers", 20011, 100, 60, "bf16", "sqeuclidean"),
    ("mixture", 2305, 8, 20, "f16", "sqeuclidean"),
    ("sorted", 70001, 17, 20, "f16", "sqeuclidean"),
    ("curves", 12345, 33, 20, "fp8", "sqeuclidean"),
    ("few", 4097, 128, 12, "fp8", "sqeuclidean"),
    ("mixture", 4100, 50, 12, "f32", "l1"),
    ("outliers", 9217, 7, 20, "f32", "l1"),
]


@pytest.mark.parametrize("data,n,d,k,dtype,dist", CASES)
def test_lists_pick_what_full_scoring_picks(data, n, d, k, dtype, dist):
    x = points(data, n, d, n)
    full, lists = both(x, k, dtype, dist)
    assert lists[0].tolist() == full[0].tolist()
    assert np.array_equal(lists[1], full[1]) and np.array_equal(lists[2], full[2])
    assert lists[3] == full[3]  # the same window


def test_lists_under_graph_replay():
    x = points("mixture", 6001, 40, 5)
    full, lists = both(x, 20, "f32", graph=True)
    assert lists[0].tolist() == full[0].tolist() and np.array_equal(lists[1], full[1])


@pytest.mark.parametrize("dtype,dist", [("f32", "sqeuclidean"), ("bf16", "sqeuclidean"), ("f32", "l1")])
def test_lists_after_other_calls(dtype, dist):
    """Gains asked for between runs use the buffers that hold the lists."""
    x = torch.from_numpy(points("mixture", 4003, 24, 7)).cuda()
    ds = ebc.Dataset(x, dtype=dtype, dist=dist)
    a = [t.cpu().numpy() for t in ds.greedy(15)]
    g0 = ds.marginal_gains().cpu().numpy()
    b = [t.cpu().numpy() for t in ds.greedy(15)]
    g1 = ds.marginal_gains().cpu().numpy()
    ds.sync()
    assert all(np.array_equal(p, q) for p, q in zip(a, b)) and np.array_equal(g0, g1)


# instances that keep lists and instances that do not, in every reduced type and float32, uneven k
BATCH = [("curves", 30000, 64, 9, "bf16"), ("mixture", 700, 16, 7, "bf16"), ("outliers", 26001, 33, 12, "fp8"),
         ("mixture", 20480, 100, 3, "f16"), ("sorted", 9000, 100, 10, "f32"), ("normal", 1500, 8, 5, "f32"),
         ("curves", 300, 500, 4, "bf16"), ("few", 24000, 128, 9, "bf16")]


@pytest.mark.parametrize("graph", [False, True])
def test_batch_with_lists_equals_solo(graph):
    dss = [ebc.Dataset(torch.from_numpy(points(*c[:3], i)).cuda(), dtype=c[4]) for i, c in enumerate(BATCH)]
    ks = [c[3] for c in BATCH]
    solo = [[t.cpu().numpy() for t in ds.greedy(k)] for ds, k in zip(dss, ks)]
    batch = ebc.Batch(dss)
    batch.set_graph(graph)
    for _ in range(2):
        got = batch.greedy(ks)
        for ds in dss:
            ds.sync()
        for a, b in zip(solo, got):
            assert all(np.array_equal(p, q.cpu().numpy()) for p, q in zip(a, b))


def test_server_with_lists_equals_solo():
    sv = ebc.Server(1 << 30, max_slots=3)
    want, ids = [], []
    for i, c in enumerate(BATCH):
        x = points(*c[:3], i)
        ds = ebc.Dataset(torch.from_numpy(x).cuda(), dtype=c[4])
        want.append([t.cpu().numpy() for t in ds.greedy(c[3])])
        ids.append(sv.submit(x, c[3], dtype=c[4]))
    for _ in range(100):
        sv.step()
        if sv.stats()["completed"] == len(ids):
            break
    for rid, w in zip(ids, want):
        r = sv.poll(rid)
        assert r["state"] == "done"
        assert np.array_equal(r["sel"], w[0]) and np.array_equal(r["f"], w[1]) and np.array_equal(r["gain"], w[2])
    sv.close()


@pytest.mark.parametrize("n", [1, 2, 255, 257, 1000, 4096, 4097])
@pytest.mark.parametrize("d,dtype", [(5, "f32"), (40, "bf16"), (200, "f32"), (131, "fp8")])
def test_small_ground_sets_equal_a_batch_of_one(n, d, dtype):
    """Solo runs on at most 4096 points take the fused stages, a batch the separate ones."""
    x = torch.from_numpy(points("few" if n == 255 else "mixture", n, d, n + d)).cuda()
    ds = ebc.Dataset(x, dtype=dtype)
    k = min(n, 11)
    solo = [t.cpu().numpy() for t in ds.greedy(k)]
    ds.sync()
    got = [t.cpu().numpy() for t in ebc.Batch([ds]).greedy([k])[0]]
    ds.sync()
    assert all(np.array_equal(a, b) for a, b in zip(solo, got))
    assert len(set(solo[0].tolist())) == k


@pytest.mark.parametrize("n,d", [(3, 4), (256, 31), (2049, 6)])
def test_small_l1_against_oracle(n, d):
    from oracle import ebc_oracle
    x = points("mixture", n, d, n)
    ds = ebc.Dataset(torch.from_numpy(x).cuda(), dist="l1")
    k = min(n, 6)
    sel, f, _ = ds.greedy(k)
    ds.sync()
    rsel, rf, _ = ebc_oracle.greedy(x, k, dist="l1")
    assert sel.cpu().numpy().tolist() == rsel.tolist()
    np.testing.assert_allclose(f.cpu().numpy(), rf, rtol=1e-12)


@pytest.mark.parametrize("n,d,dtype,k", [(300, 129, "f32", 12), (1000, 777, "f32", 20), (1000, 777, "bf16", 20),
                                         (513, 400, "f16", 9), (4096, 150, "fp8", 15), (4097, 150, "f32", 6)])
def test_pair_matrix_picks_what_dot_products_pick(n, d, dtype, k):
    """Long rows: a profiled run multiplies the rows at every step; a workspace
    without room for the pair matrix makes every run do so."""
    x = points("curves", n, d, n + d)
    full, matrix = both(x, k, dtype)
    assert matrix[0].tolist() == full[0].tolist()
    assert np.array_equal(matrix[1], full[1]) and np.array_equal(matrix[2], full[2])
    t = torch.from_numpy(x).cuda()
    lib, nbytes = ebc.lib(), ebc.Dataset(t, dtype=dtype).workspace_bytes
    n_pad = -(-n // 256) * 256
    least = nbytes - (4 * n_pad * n_pad if n <= 4096 else 0)
    ds = ebc.Dataset.__new__(ebc.Dataset)
    ds.x, ds.n, ds.d, ds.dtype, ds.dist, ds._h = t, n, d, dtype, "sqeuclidean", None
    ds.workspace = torch.empty(least, dtype=torch.uint8, device="cuda")
    import ctypes
    h = ctypes.c_void_p()
    args = (ctypes.c_void_p(t.data_ptr()), n, d, ebc.DTYPES[dtype], 0, ctypes.c_void_p(ds.workspace.data_ptr()))
    stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    assert lib.ebc_dataset_create(*args, least - 1, stream, ctypes.byref(h)) == 1  # invalid argument, as before
    assert lib.ebc_dataset_create(*args, least, stream, ctypes.byref(h)) == 0
    ds._h = h
    sel, f, _ = ds.greedy(k)
    ds.sync()
    assert sel.cpu().numpy().tolist() == full[0].tolist() and np.array_equal(f.cpu().numpy(), full[1])
    got = [q.cpu().numpy() for q in ebc.Batch([ebc.Dataset(t, dtype=dtype), ds]).greedy([k, k])[0]]
    assert np.array_equal(got[0], full[0]) and np.array_equal(got[1], full[1])


@pytest.mark.parametrize("n,d,dtype", [(5003, 100, "f32"), (700, 9, "f32"), (40000, 24, "f32"), (20011, 128, "f32"),
                                       (9001, 33, "bf16"), (33000, 128, "f16"), (4000, 128, "fp8")])
def test_gains_of_lists_of_every_length(n, d, dtype):
    """Lists take another kernel by their length: the same gains as of all points, bit for bit."""
    x = torch.from_numpy(points("mixture", n, d, n)).cuda()
    ds = ebc.Dataset(x, dtype=dtype)
    ds.greedy(3)
    full = ds.marginal_gains().cpu().numpy()
    rng = np.random.default_rng(n)
    for c in (1, 31, 32, 33, 129, 257, 513, 2303, n - 1, n, n + 300):
        cand = rng.integers(0, n, c).astype(np.int32)
        got = ds.marginal_gains(cand=torch.from_numpy(cand)).cpu().numpy()
        assert np.array_equal(got, full[cand]), c
    ds.sync()
