"""The sweep with several lines per wave where it can go wrong: frequency counts and blocks around
its lanes (V values each), its lines per wave and its chunks of lanes; shifts far beyond a block on
both sides; lines of the origin alone; every schedule.  A plan of a moving model reads padded tables
there while rt_solve sweeps one line per wave: the same operations, so J is equal bit for bit; static
models and plans alike are held to the oracle by the bars of the FP64 and FP32 sweeps."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

TOL = {True: 1e-12, False: 1e-4}  # relative, FP64 and FP32 sweeps (as for every second-order sweep)

# lengths of the frequency blocks, their widths (equal or not)
BLOCKS = [([1], [0.5]), ([2], [0.5]), ([3], [0.5]), ([5], [0.5]), ([17], [0.5]), ([31], [0.5]), ([64], [0.5]),
          ([65], [0.5]), ([48, 48], [0.5, 0.5]), ([1, 7, 2, 12], [0.5, 0.5, 0.5, 0.5]), ([12, 9], [0.5, 0.6]),
          ([130], [0.25]), ([255], [0.1]), ([259], [0.1]), ([200, 130], [0.1, 0.1]), ([300, 211], [0.1, 0.12])]


def _model(lens, dx, moving):
    m = synth.tiny_model(300 + sum(lens), P=70, F=sum(lens), moving=moving)
    m.freq = synth.FreqGrid(np.array(lens, np.int32), np.full(len(lens), -2.0), np.array(dx))
    if moving:  # shifts of a fraction of a cell up to far past the longest block
        rng = np.random.default_rng(sum(lens))
        m.vel[:] = m.vel * 10.0 ** rng.uniform(-2, 2.5, (m.P, 1))
    return m


@pytest.mark.parametrize("blocks", BLOCKS, ids=lambda b: "+".join(map(str, b[0])))
@pytest.mark.parametrize("moving", [True, False])
@pytest.mark.parametrize("fp64", [True, False])
def test_lines(rt, orc, blocks, moving, fp64):
    import torch
    m = _model(*blocks, moving)
    prec = rt.RT_F64 if fp64 else rt.RT_F32
    dt = torch.float64 if fp64 else torch.float32
    c32, e32, c64, e64 = synth.to_fp32_tables(m.chi, m.eta)
    model = rt.Model.from_numpy(m.pos, m.nbr_off, m.nbr_idx, m.vel)
    ds = rt.DirSet.uniform(2)
    _, dirs, w2 = orc.dirset_uniform(2)
    org = torch.arange(m.P, dtype=torch.int32, device="cuda")
    chi = torch.as_tensor(c64, device="cuda").to(dt)
    eta = torch.as_tensor(e64, device="cuda").to(dt)
    I_bc = torch.as_tensor(m.I_bc, dtype=torch.float64, device="cuda")
    one = rt.solve(model, ds, rt.trace(model, ds, origins=org), chi, eta, m.freq.len, m.freq.dx, I_bc, origins=org,
                   precision=prec).cpu().numpy()
    Je = orc.compute_J(m, dirs, w2, origins=org.cpu().numpy(), chi=c64, eta=e64)
    assert np.max(np.abs(one - Je) / np.abs(Je)) <= TOL[fp64]
    for schedule in (rt.SCHED_DIRECT, rt.SCHED_SPATIAL, rt.SCHED_BINNED):
        J = torch.empty((m.P, m.F), dtype=dt, device="cuda")
        plan = rt.Plan(model, ds, chi, eta, m.freq.len, m.freq.dx, I_bc, J, origins=org, precision=prec,
                       schedule=schedule)
        plan.run()
        rt.sync_status()
        assert plan.rays()[1].numel() >= 32 * m.P  # enough line points for the padded tables
        assert np.array_equal(J.cpu().numpy(), one), schedule
