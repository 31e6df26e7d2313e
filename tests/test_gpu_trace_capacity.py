"""Lists that do not fit: rt_trace fills what it has room for with the lists' own entries, reports the
total and latches the error; and its write pass does not go on along rays that it can no longer store."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("model", ["tiny", "lattice"])
@pytest.mark.parametrize("capacity", [0, 1, 7, 8, 9, 15, 16, 17, 1000, -1])
def test_truncated_lists(rt, model, capacity):
    """Capacities around the blocks of eight entries that lists are stored in; -1: one entry short."""
    m = synth.tiny_model(12, P=70) if model == "tiny" else synth.lattice_model(7)
    gm = rt.Model.from_numpy(m.pos, m.nbr_off, m.nbr_idx, m.vel)
    ds = rt.DirSet.uniform(1)
    off, ids, Z = rt.trace(gm, ds, n_origins=m.P)
    n = ids.numel()
    cap = n - 1 if capacity < 0 else capacity
    assert cap < n
    off2, ids2, Z2, total = rt.trace_once(gm, ds, cap, n_origins=m.P)
    with pytest.raises(rt.RtError):
        rt.sync_status()
    assert total == n
    assert np.array_equal(off2.cpu().numpy(), off.cpu().numpy())
    assert np.array_equal(ids2[:cap].cpu().numpy(), ids[:cap].cpu().numpy())
    assert np.array_equal(Z2[:cap].cpu().numpy(), Z[:cap].cpu().numpy())
    rt.sync_status()


def test_no_room_costs_the_count_only(rt):
    """Rays of some 2000 entries along a chain of points: with room for one entry the write pass ends after
    eight steps, so the call takes little more than its count pass, about half of the whole lists' time."""
    import torch
    rng = np.random.default_rng(13)
    P = 4000
    pos = np.stack([np.arange(P) + rng.uniform(-0.2, 0.2, P), *rng.uniform(-0.2, 0.2, (2, P))], 1)
    off, idx = synth.models.csr_from_edges(P, np.arange(P - 1), np.arange(1, P))
    gm = rt.Model.from_numpy(pos, off, idx, None)
    ds = rt.DirSet.uniform(1)
    org = torch.arange(0, P, 50, dtype=torch.int32, device="cuda")
    n = rt.trace(gm, ds, origins=org)[1].numel()
    assert n > 500 * org.numel() * 2 * ds.R
    t = []
    for cap in (1, n):
        best = np.inf
        for _ in range(5):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            rt.trace_once(gm, ds, cap, origins=org)
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b))
        t.append(best)
    with pytest.raises(rt.RtError):
        rt.sync_status()
    print("ms:", t)
    assert t[0] <= 0.75 * t[1]
