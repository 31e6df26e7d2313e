"""Rows of a model with a hub: a point that has every other as its neighbour is laid out in time
proportional to its row when the row is given in order, and rows in any order give the same lists."""
import time

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


def test_hub_row_time(rt):
    """100 000 neighbours of one point: a model of milliseconds (each entry against each would be 1e10)."""
    import torch
    P = 100_001
    rng = np.random.default_rng(31)
    pos = rng.normal(size=(P, 3))
    off, idx = synth.models.csr_from_edges(P, np.zeros(P - 1, np.int64), np.arange(1, P))
    small = synth.tiny_model(32)
    rt.Model.from_numpy(small.pos, small.nbr_off, small.nbr_idx, None)  # the library's code is on the device
    torch.cuda.synchronize()
    t = time.perf_counter()
    model = rt.Model.from_numpy(pos, off, idx, None)
    t = time.perf_counter() - t
    print(f"{t * 1e3:.1f} ms")
    off_r, ids, Z = (x.cpu().numpy() for x in rt.trace(model, rt.DirSet.uniform(1),
                                                        origins=torch.tensor([5], dtype=torch.int32, device="cuda")))
    for s in range(len(off_r) - 1):  # from a leaf to the hub, if it is forward, and on to another leaf
        assert off_r[s + 1] - off_r[s] <= 2
        if off_r[s + 1] > off_r[s]:
            assert ids[off_r[s]] == 0
    assert t < 1.0


@pytest.mark.parametrize("order", ["reversed", "shuffled"])
def test_rows_in_any_order(rt, order):
    m = synth.tiny_model(33, P=120)
    rng = np.random.default_rng(34)
    idx = m.nbr_idx.copy()
    for p in range(m.P):
        row = idx[m.nbr_off[p]:m.nbr_off[p + 1]]
        row[:] = row[::-1] if order == "reversed" else rng.permutation(row)
    ds = rt.DirSet.uniform(2)
    a, b = (rt.trace(rt.Model.from_numpy(m.pos, m.nbr_off, i, None), ds, n_origins=m.P) for i in (m.nbr_idx, idx))
    for x, y in zip(a, b):
        assert np.array_equal(x.cpu().numpy(), y.cpu().numpy())
