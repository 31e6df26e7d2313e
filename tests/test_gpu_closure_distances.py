"""The mean neighbour distance of the closure's features, at the numbers of frequencies where the workgroup's
points change from a wave each to groups of 16, 8 and 4 lanes to a thread each, over rows of 1 to 150 entries."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def cloud():
    """700 points, degrees 1 to 150 in no order."""
    rng = np.random.default_rng(41)
    P = 700
    pos = rng.normal(size=(P, 3))
    want = rng.integers(1, 76, P)
    a = np.repeat(np.arange(P), want)
    b = rng.integers(0, P - 1, len(a))
    b += b >= a
    key = np.unique(np.minimum(a, b) * P + np.maximum(a, b))
    off, idx = synth.models.csr_from_edges(P, key // P, key % P)
    L = np.empty(P, np.float32)
    for p in range(P):
        s = 0.0
        for d in np.sqrt(((pos[idx[off[p]:off[p + 1]]] - pos[p]) ** 2).sum(1)):
            s += d
        L[p] = s / (off[p + 1] - off[p])
    return pos, off, idx, L


@pytest.mark.parametrize("F", [1, 2, 3, 4, 5, 7, 8, 9, 15, 16, 17, 28, 31, 32, 33, 40, 64])
@pytest.mark.parametrize("subset", [False, True])
def test_mean_distance(rt, cloud, F, subset):
    import torch
    pos, off, idx, L = cloud
    P = len(L)
    rng = np.random.default_rng(F)
    model = rt.Model.from_numpy(pos, off, idx, None)
    chi = torch.from_numpy(rng.uniform(0.1, 1.0, (P, F)).astype(np.float32)).cuda()
    pts = rng.permutation(P)[: P - 13].astype(np.int32) if subset else np.arange(P, dtype=np.int32)
    J1 = torch.from_numpy(rng.uniform(0.1, 1.0, (len(pts), F)).astype(np.float32)).cuda()
    fx = torch.linspace(-5, 5, F, device="cuda")
    feat = rt.closure_features(model, chi, 0.5 * chi, fx, J1, points=torch.from_numpy(pts).cuda() if subset else None)
    got = feat.cpu().numpy().reshape(len(pts), F, 16)[:, :, 8]
    want = np.log(L[pts].astype(np.float64))
    # one rounding of the mean to FP32 on both sides, the sum in any order, and FP32's logarithm
    assert np.all(np.abs(got - want[:, None]) <= 2.0**-22 + 2.0**-22 * np.abs(want[:, None]))
