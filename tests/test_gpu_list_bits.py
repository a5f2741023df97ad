"""Greedy steps that score a list of candidates (csrc/lazy.h) at sizes where solo
runs, batches and the server do: the picks, f and gains of a run that scores every
candidate at every step (profiling on), bit for bit, also where more candidates come
near the best than are re-scored. Every case asserts that its runs scored lists."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2105_12026_amd import ebc, workloads

pytestmark = pytest.mark.gpu


def points(data, n, d, seed):
    rng = np.random.default_rng([17, seed])
    if data == "curves":
        return workloads.process_curves(rng, n, d).astype(np.float32)
    if data == "normal":
        return rng.standard_normal((n, d)).astype(np.float32)
    if data == "near":  # 6 points, each repeated with small noise: thousands of gains within rounding of the best
        x = workloads.gaussian_mixture(rng, 6, d, 6)[rng.integers(0, 6, n)]
        return (x + 1e-3 * rng.standard_normal((n, d))).astype(np.float32)
    if data == "tied":  # 1024-point cubes around centres of falling norm: a cube's gains are equal, its float32 sums not
        centres = -(-n // 1024)
        cube = 37.0 * (1 - 2 * ((np.arange(1024)[:, None] >> np.arange(10)) & 1))
        x = np.zeros((centres * 1024, 10 + centres))
        for i in range(centres):
            x[i * 1024:(i + 1) * 1024, :10] = cube
            x[i * 1024:(i + 1) * 1024, 10 + i] = round(600 * 1.1 ** i)
        assert x.shape == (n, d)
        return x[rng.permutation(n)].astype(np.float32)
    x = workloads.gaussian_mixture(rng, n, d, 12)
    if data == "few":  # 7 distinct points: after 7 picks every gain is 0
        x = x[rng.integers(0, 7, n)]
    return x.astype(np.float32)


def stats(ds):
    st = ebc._Stats()
    stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    assert ebc.lib().ebc_sync_status(ds.handle, stream, ctypes.byref(st)) == 0
    return st


def host(out):
    return [q.cpu().numpy() for q in out]


def same(a, b):
    return all(np.array_equal(p, q) for p, q in zip(a, b))


def full_run(t, k, dtype, dist="sqeuclidean"):
    ds = ebc.Dataset(t, dtype=dtype, dist=dist)
    ds.profile(True)
    out = host(ds.greedy(k))
    st = stats(ds)
    assert st.list_steps == 0
    return out, st


# (data, n, d, k, dtype, dist, least window_max of the full run)
SOLO = [("near", 12003, 16, 20, "f32", "sqeuclidean", 1025), ("near", 9217, 100, 20, "f32", "sqeuclidean", 1025),
        ("near", 20011, 64, 20, "bf16", "sqeuclidean", 1025), ("near", 16500, 100, 20, "f16", "sqeuclidean", 1025),
        ("near", 30011, 33, 20, "fp8", "sqeuclidean", 1025), ("near", 10007, 50, 20, "f32", "l1", 1025),
        ("tied", 12288, 22, 10, "f32", "sqeuclidean", 1023), ("tied", 21504, 31, 12, "bf16", "sqeuclidean", 1023),
        ("tied", 21504, 31, 12, "f16", "sqeuclidean", 1023), ("tied", 21504, 31, 12, "fp8", "sqeuclidean", 1023),
        ("few", 11001, 20, 12, "f32", "sqeuclidean", 1025), ("few", 26003, 128, 12, "fp8", "sqeuclidean", 1025),
        ("few", 9001, 30, 12, "f32", "l1", 1025), ("curves", 24001, 33, 20, "fp8", "sqeuclidean", 0),
        ("mixture", 17001, 64, 30, "bf16", "sqeuclidean", 0), ("mixture", 33001, 3, 25, "f32", "sqeuclidean", 0)]


@pytest.mark.parametrize("data,n,d,k,dtype,dist,window", SOLO)
def test_solo(data, n, d, k, dtype, dist, window):
    t = torch.from_numpy(points(data, n, d, n)).cuda()
    want, full = full_run(t, k, dtype, dist)
    assert full.window_max >= window
    ds = ebc.Dataset(t, dtype=dtype, dist=dist)
    assert same(host(ds.greedy(k)), want)
    st = stats(ds)
    assert st.list_steps == k - 1
    if window:
        assert (st.window_max, st.window_overflow) == (full.window_max, full.window_overflow)


@pytest.mark.parametrize("data,n,d,dtype", [("mixture", 9217, 40, "f32"), ("near", 16411, 64, "bf16")])
def test_graph_replays(data, n, d, dtype):
    """Each replay reads the list's sizes on the device; other work in between."""
    t = torch.from_numpy(points(data, n, d, 5)).cuda()
    k = 15
    want, _ = full_run(t, k, dtype)
    ds = ebc.Dataset(t, dtype=dtype)
    ds.set_graph(True)
    outs = [torch.empty(k, dtype=q, device="cuda") for q in (torch.int32, torch.float64, torch.float64)]
    e0 = torch.full((d,), 0.5, device="cuda")
    for i in range(4):
        got = host(ds.greedy(k, sel=outs[0], f=outs[1], gain=outs[2]))
        assert same(got, want) and stats(ds).list_steps == k - 1
        if i == 1:  # a replay over other minima, and back
            ds.set_e0(e0)
            eager = ebc.Dataset(t, dtype=dtype)
            eager.set_e0(e0)
            assert same(host(ds.greedy(k, sel=outs[0], f=outs[1], gain=outs[2])), host(eager.greedy(k)))
            ds.set_e0(None)
        ds.marginal_gains()


@pytest.mark.parametrize("n,d,dtype,dist", [(10241, 24, "f32", "sqeuclidean"), (17003, 64, "bf16", "sqeuclidean"),
                                            (8003, 24, "f32", "l1")])
def test_calls_between_runs(n, d, dtype, dist):
    """Gains asked for between runs use buffers of the runs."""
    t = torch.from_numpy(points("mixture", n, d, 7)).cuda()
    want, _ = full_run(t, 15, dtype, dist)
    ds = ebc.Dataset(t, dtype=dtype, dist=dist)
    gains = []
    for _ in range(2):
        assert same(host(ds.greedy(15)), want) and stats(ds).list_steps == 14
        gains.append(ds.marginal_gains().cpu().numpy())
    assert np.array_equal(*gains)


# large and small instances of one row padding: those lists are worth it for, and those they are not
MIXED = {"bf16": [("mixture", 30000, 64), ("near", 1024, 64), ("mixture", 2305, 60), ("near", 9000, 64)],
         "f32": [("mixture", 12000, 96), ("near", 700, 96), ("mixture", 4097, 90), ("near", 5003, 96)],
         "fp8": [("curves", 30000, 64), ("near", 1500, 50), ("near", 12345, 33), ("normal", 6000, 64)],
         "f16": [("near", 30000, 32), ("near", 7000, 32), ("few", 3000, 30), ("mixture", 11000, 20)]}


@pytest.mark.parametrize("dtype", sorted(MIXED))
@pytest.mark.parametrize("graph", [False, True])
def test_mixed_batch(dtype, graph):
    ts = [torch.from_numpy(points(*c, i)).cuda() for i, c in enumerate(MIXED[dtype])]
    ks = [11, 7, 14, 12]
    want = [full_run(t, k, dtype)[0] for t, k in zip(ts, ks)]
    dss = [ebc.Dataset(t, dtype=dtype) for t in ts]
    batch = ebc.Batch(dss)
    batch.set_graph(graph)
    for _ in range(2):
        got = [host(g) for g in batch.greedy(ks)]
        listed = [stats(ds).list_steps for ds in dss]
        assert all(same(g, w) for g, w in zip(got, want))
        assert listed[0] == ks[0] - 1
    solo = [host(ds.greedy(k)) for ds, k in zip(dss, ks)]
    assert all(same(g, w) for g, w in zip(solo, want))


@pytest.mark.parametrize("dtype", sorted(MIXED))
def test_mixed_requests(dtype):
    """Served alone and together: lists start, and end, while a request runs."""
    xs = [points(*c, i) for i, c in enumerate(MIXED[dtype])]
    ks = [11, 7, 14, 12]
    want = [full_run(torch.from_numpy(x).cuda(), k, dtype)[0] for x, k in zip(xs, ks)]
    for alone in (False, True):
        sv = ebc.Server(1 << 30, max_slots=1 if alone else 4)
        ids = []
        for x, k in zip(xs[::-1], ks[::-1]):  # the large one joins last
            ids.insert(0, sv.submit(x, k, dtype=dtype))
            sv.step()
        for _ in range(sum(ks) + 8):
            sv.step()
        for rid, w in zip(ids, want):
            r = sv.poll(rid)
            assert r["state"] == "done" and same([r[q] for q in ("sel", "f", "gain")], w)
        sv.close()


@pytest.mark.parametrize("data,n,d,dtype", [("near", 4096, 16, "f32"), ("near", 1400, 30, "bf16"),
                                            ("few", 3999, 20, "fp8"), ("few", 1300, 9, "f16")])
def test_window_overflow_of_small_ground_sets(data, n, d, dtype):
    """The fused stages of a small solo run and the separate ones of a batch keep the same candidates."""
    t = torch.from_numpy(points(data, n, d, n)).cuda()
    ds = ebc.Dataset(t, dtype=dtype)
    solo = host(ds.greedy(12))
    st = stats(ds)
    assert st.window_overflow > 0 and st.list_steps == 0
    batch = host(ebc.Batch([ds]).greedy([12])[0])
    assert same(batch, solo) and stats(ds).window_overflow == st.window_overflow
