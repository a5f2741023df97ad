"""A batch whose gains launch has more than 2^24 workgroups (2^32 threads, more than
one launch can have): every instance gets its solo result."""
import pytest
import torch

from paper_2105_12026_amd import ebc

pytestmark = pytest.mark.gpu


def test_more_workgroups_than_a_launch_has():
    x = torch.randn(4000, 5, device="cuda", generator=torch.Generator(device="cuda").manual_seed(3))
    one = ebc.Dataset(x)
    k = 2
    solo = [q.cpu() for q in one.greedy(k)]
    per = ebc.Batch([one]).info()["gains_workgroups_per_tick"]
    count = (1 << 24) // per + 464
    batch = ebc.Batch([ebc.Dataset(x) for _ in range(count)])
    assert batch.info()["gains_workgroups_per_tick"] > 1 << 24
    outs = [torch.zeros((count, k), dtype=t, device="cuda") for t in (torch.int32, torch.float64, torch.float64)]
    batch.greedy([k] * count, outs=list(zip(*outs)))
    for got, want in zip(outs, solo):
        assert bool((got.cpu() == want).all())
