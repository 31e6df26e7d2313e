"""The features, their normalisation and the closure's assembly over the shapes their kernels tell
apart: frequency counts around the lanes of a point and the points of a workgroup, points with more
neighbours than are kept, arrays that are not 16-byte aligned.  The features are held to a plain
FP64 reference (means of up to 69 FP32 logarithms of order 1: 69/2 x 2^-24 x a few is below 1e-5),
the aligned and unaligned paths to each other bit for bit."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


def _model(F):
    m = synth.tiny_model(500 + F, P=70, F=F)
    hub = np.setdiff1d(np.arange(1, 70), m.nbr_idx[m.nbr_off[0]:m.nbr_off[1]])  # point 0: everyone's neighbour
    src = np.repeat(np.arange(70), np.diff(m.nbr_off))
    a = np.concatenate([src, np.zeros_like(hub), hub])
    b = np.concatenate([m.nbr_idx, hub, np.zeros_like(hub)])
    o = np.lexsort((b, a))
    m.nbr_off = np.concatenate([[0], np.cumsum(np.bincount(a, minlength=70))]).astype(m.nbr_off.dtype)
    m.nbr_idx = b[o].astype(m.nbr_idx.dtype)
    return m


@pytest.mark.parametrize("F", [1, 3, 31, 32, 40, 64, 65, 300])
def test_shapes(rt, F):
    import torch
    m = _model(F)
    model = rt.Model.from_numpy(m.pos, m.nbr_off, m.nbr_idx, None)
    rng = np.random.default_rng(F)
    R = 25 if F < 40 else 6
    f32 = lambda a: torch.as_tensor(np.asarray(a, np.float32), device="cuda")
    chi, eta, J1, u, x = f32(m.chi), f32(m.eta), f32(rng.uniform(.2, 2, (70, F))), \
        f32(rng.uniform(.1, 3, (70, R, F))), f32(np.linspace(-4, 4, F))
    n = 70 * F
    buf = torch.empty(n * 16 + 4, dtype=torch.float32, device="cuda")
    got = [rt.closure_features(model, chi, eta, x, J1, u=u, feat=buf[s:s + n * 16].view(n, 16)).clone() for s in (0, 1)]
    assert torch.equal(got[0], got[1])
    c, S, J, U = (t.double().cpu().numpy() for t in (chi, eta / chi, J1, u))
    ref = np.zeros((70, F, 16))
    a = np.log(U) - np.log(J)[:, None]
    for p in range(70):
        q = m.nbr_idx[m.nbr_off[p]:m.nbr_off[p + 1]]
        L = np.mean(np.linalg.norm(m.pos[q] - m.pos[p], axis=1))
        cols = [np.log(J[p]), np.log(c[p]), np.log(S[p]), np.log(c[q]).mean(0), np.log(S[q]).mean(0), np.log(c[q]).std(0),
                np.abs((c[p] - c[q]) / (c[p] + c[q])).max(0), np.abs((S[p] - S[q]) / (S[p] + S[q])).max(0),
                np.full(F, np.log(L)), np.log(c[p] * L), x.double().cpu().numpy() / 5, np.full(F, np.log(len(q))),
                a[p].max(0), a[p].min(0), a[p].std(0)]
        ref[p, :, :15] = np.stack(cols, 1)
    assert np.max(np.abs(got[0].double().cpu().numpy().reshape(70, F, 16) - ref)) <= 1e-5
    mean, istd = rng.normal(size=16).astype(np.float32), rng.uniform(.5, 2, 16).astype(np.float32)
    xb = torch.empty(n * 16 + 8, dtype=torch.int16, device="cuda")
    X = [rt.closure_normalize(got[0], mean, istd, X=xb[s:s + n * 16].view(n, 16)).clone() for s in (0, 1)]
    want = ((got[0] - f32(mean)) * f32(istd)).to(torch.bfloat16).view(torch.int16)
    assert torch.equal(X[0], want) and torch.equal(X[1], want)
    Y = f32(rng.normal(0, .5, (n, 2)))
    Jc, fl, k = rt.closure_apply(J1, Y, 0.6)
    torch.cuda.synchronize()
    hot = torch.nonzero((0.5 * Y[:, 1].view(70, F) > 0.6).any(1)).flatten().cpu().numpy()
    k = int(k.item()) if torch.is_tensor(k) else int(k)
    assert np.array_equal(np.sort(fl.cpu().numpy()[:k]), hot)
    r = (J1.double() * torch.exp(Y[:, 0].double()).view(70, F)).cpu().numpy()
    assert np.max(np.abs(Jc.cpu().numpy() - r) / r) <= 1e-6  # exp in FP32 and one product
