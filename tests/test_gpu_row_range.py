"""FP32 second-order rows at the ends of their range: points of opacity 1e4 and more (per unit
length) among points of 1e-35, as a thick cell beside an empty one or a line's far wing, in lengths of
order one and of 1e21, and with no emission at all.  J of every path that takes the row (static
and moving plans, rt_solve, lines refined by optical depth and by velocity) is held to the FP64
oracle by the bar of the FP32 sweeps: all terms are positive, so a value that stays in range is
good to some 1e-6."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

TOL32 = 1e-4


def _model(kind, moving):
    m = synth.tiny_model(410, P=70, F=9, moving=moving)
    rng = np.random.default_rng(411)
    wall = rng.random(m.P) < 0.3
    thick = np.full(m.P, 1e4) if kind == "dark" else 10.0 ** rng.uniform(4, 8, m.P)
    m.chi = np.where(wall, thick, 1e-35)[:, None] * rng.uniform(0.5, 2.0, (m.P, m.F))
    m.eta = m.chi * rng.uniform(0.1, 2.0, (m.P, m.F)) * (0.0 if kind == "dark" else 1.0)
    m.I_bc[:] = 0.5
    if kind == "long":  # the same depths of the thick points; thin ones of 1e-36 over 1e21
        m.pos = m.pos * 1e21
        f = np.where(wall, 1e-21, 0.1)[:, None]
        m.chi, m.eta = m.chi * f, m.eta * f
    return m


@pytest.mark.parametrize("path", ["plan", "solve", "dtau", "dv"])
@pytest.mark.parametrize("kind", ["unit", "long", "dark"])
@pytest.mark.parametrize("moving", [False, True])
def test_row_range(rt, orc, kind, moving, path):
    import torch
    m = _model(kind, moving or path == "dv")
    c32, e32, c64, e64 = synth.to_fp32_tables(m.chi, m.eta)
    model = rt.Model.from_numpy(m.pos, m.nbr_off, m.nbr_idx, m.vel)
    ds = rt.DirSet.uniform(2)
    _, dirs, w2 = orc.dirset_uniform(2)
    org = torch.arange(m.P, dtype=torch.int32, device="cuda")
    chi, eta = (torch.as_tensor(x, device="cuda") for x in (c32, e32))
    I_bc = torch.as_tensor(m.I_bc, dtype=torch.float64, device="cuda")
    ref = {"dtau": dict(dtau_max=1e6), "dv": dict(dv_max=2.0)}.get(path, {})
    if path == "plan":
        J = torch.empty((m.P, m.F), dtype=torch.float32, device="cuda")
        rt.Plan(model, ds, chi, eta, m.freq.len, m.freq.dx, I_bc, J, origins=org, schedule=rt.SCHED_SPATIAL).run()
    else:
        J = rt.solve(model, ds, rt.trace(model, ds, origins=org), chi, eta, m.freq.len, m.freq.dx, I_bc, origins=org,
                     **ref)
    rt.sync_status()
    Je = orc.compute_J(m, dirs, w2, origins=org.cpu().numpy(), chi=c64, eta=e64, **ref)
    assert np.max(np.abs(J.cpu().numpy() - Je) / Je) <= TOL32
