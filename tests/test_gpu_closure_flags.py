"""Flagged points of the closure: each once whatever the widths, and counted without one atomic per point."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _inputs(n, F, share, seed):
    """J1, Y and the flagged points for a bound of 1: predicted log-variance 4 at one frequency of each, else 0."""
    rng = np.random.default_rng(seed)
    J1 = rng.uniform(0.5, 2.0, (n, F)).astype(np.float32)
    Y = np.zeros((n, F, 2), np.float32)
    Y[..., 0] = rng.uniform(-1, 1, (n, F))
    want = np.nonzero(rng.random(n) < share)[0]
    Y[want, rng.integers(0, F, len(want)), 1] = 4.0
    return J1, Y.reshape(n * F, 2), want


@pytest.mark.parametrize("F", [1, 2, 3, 4, 16, 33, 64, 65, 200])
@pytest.mark.parametrize("n", [1, 63, 257, 4099, 70001])
def test_each_flagged_point_once(rt, n, F):
    import torch
    if n * F > 5_000_000:
        n = 5_000_000 // F
    for share in (0.0, 0.3, 1.0):
        J1, Y, want = _inputs(n, F, share, 7 * n + F)
        J, fl, k = rt.closure_apply(torch.from_numpy(J1).cuda(), torch.from_numpy(Y).cuda(), 1.0)
        k = int(k.item())
        assert k == len(want)
        assert np.array_equal(np.sort(fl.cpu().numpy()[:k]), want)
        # J1 e^Y in FP32: half an ulp of the product, and the fast exponential's few
        np.testing.assert_allclose(J.cpu().numpy(), J1 * np.exp(Y[:, 0].reshape(n, F).astype(np.float64)), rtol=2e-6)


@pytest.mark.parametrize("F", [64, 16])
def test_flagging_every_point_costs_little(rt, F):
    """65 536 flags by one atomic each wait for one another for several times the pass over J."""
    import torch
    n = 65536
    times = []
    for share in (0.0, 1.0):
        J1, Y, _ = _inputs(n, F, share, 5)
        J1, Y = torch.from_numpy(J1).cuda(), torch.from_numpy(Y).cuda()
        for _ in range(3):
            rt.closure_apply(J1, Y, 1.0)
        best = np.inf
        for _ in range(10):
            t0, t1 = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            t0.record()
            for _ in range(4):
                rt.closure_apply(J1, Y, 1.0)
            t1.record()
            t1.synchronize()
            best = min(best, t0.elapsed_time(t1) / 4)
        times.append(best)
    print(f"none {times[0] * 1e3:.1f} us, all {times[1] * 1e3:.1f} us")
    # some hundred additions and the list's 256 kB beside 16 to 67 MB
    assert times[1] < 1.5 * times[0] + 0.01
