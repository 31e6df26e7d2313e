"""The fused training step and the small-batch forward at the edges of their tiles: a captured step
equals the same step called piece by piece bit for bit (its loss the FP64 sum of the samples' to
rounding), and a
sample's output does not depend on the batch, the tile width or the lane it falls on."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _data(n):
    import torch
    rng = np.random.default_rng(n)
    X = torch.as_tensor(rng.normal(size=(n, 16)).astype(np.float32)).to(torch.bfloat16).view(torch.int16).cuda()
    return X, torch.as_tensor(rng.normal(0.0, 0.5, n).astype(np.float32)).cuda()


def _rows(seed, k, batch, n):
    i = (np.uint64(k) * np.uint64(batch) + np.arange(1, batch + 1, dtype=np.uint64))
    with np.errstate(over="ignore"):
        z = np.uint64(seed) + i * np.uint64(0x9E3779B97F4A7C15)
        z = (z ^ (z >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
        z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
        z ^= z >> np.uint64(31)
    return (z % np.uint64(n)).astype(np.int32)


@pytest.mark.parametrize("batch", [1, 31, 32, 33, 8192, 8193, 65535, 65536])
def test_step_equals_its_pieces(rt, batch):
    import torch
    X, T = _data(5000)
    a, b = rt.MLP(seed=4), rt.MLP(seed=4)
    la, loss = torch.zeros(1, dtype=torch.float32, device="cuda"), 0.0
    # lr_final = lr: the rate of every step is lr
    a.train(X, T, 2, batch=batch, total_steps=5, lr=1e-3, lr_final=1e-3, wd=1e-3, seed=9, loss_sum=la)
    for k in range(2):
        rows = torch.as_tensor(_rows(9, k, batch, 5000)).cuda()
        Y = b.forward(X, rows=rows, keep=True)
        dY = rt.mlp_nll(Y, T, rows=rows)
        m, s, t = Y[:, 0].double(), Y[:, 1].double(), T[rows.long()].double()
        loss += float((0.5 * (torch.exp(-s) * (t - m) ** 2 + s)).sum())
        b.zero_grad()
        b.backward(X, dY, rows=rows)
        b.adam_step(lr=float(np.float32(1e-3)), wd=1e-3)
    assert np.array_equal(a.get_params(), b.get_params())
    assert np.array_equal(a.get_grads(), b.get_grads())
    # the published copies serve the next forward: the same output from both
    assert torch.equal(a.forward(X), b.forward(X))
    # n terms of order 1 summed in trees and added once per step, FP32
    if batch < 65536:  # from there on the loss is the separate kernel's
        assert abs(la.item() - loss) <= 2.0 ** -22 * batch * 2


@pytest.mark.parametrize("n", [1, 17, 33, 65, 8192, 8193, 40001])
def test_forward_does_not_depend_on_the_batch(rt, n):
    import torch
    X, _ = _data(n)
    net = rt.MLP(seed=6)
    Y = net.forward(X)
    perm = torch.randperm(n, device="cuda", dtype=torch.int64)
    assert torch.equal(net.forward(X, rows=perm.to(torch.int32)), Y[perm])
    assert torch.equal(net.forward(X[: (n + 1) // 2].contiguous(), keep=True), Y[: (n + 1) // 2])
