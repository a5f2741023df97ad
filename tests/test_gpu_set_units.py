"""Set indices are checked by eight lanes a set (ebc_eval_sets)."""
import numpy as np
import pytest
import torch

from paper_2105_12026_amd import ebc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("size", [1, 7, 8, 9, 16, 149])
def test_a_set_index_out_of_range_is_found_anywhere(size):
    """Eight lanes read a set's indices: a bad one in the first, last or any
    other place of the last, partial, round is an error; none is not."""
    x = torch.from_numpy(np.random.default_rng(3).standard_normal((300, 12)).astype(np.float32)).cuda()
    sets = 5
    off = torch.arange(sets + 1, dtype=torch.int64) * size
    good = torch.arange(sets * size, dtype=torch.int32) % 300
    print(f"[gpu-case] eval_sets bad index, sets of {size}", flush=True)
    ds = ebc.Dataset(x)
    ds.eval_sets(off, good)
    ds.sync()
    for at in sorted({0, size // 2, size - 1}):
        idx = good.clone()
        idx[3 * size + at] = 300 if at else -1
        ds = ebc.Dataset(x)
        with pytest.raises(ebc.EBCError):
            ds.eval_sets(off, idx)
            ds.sync()
