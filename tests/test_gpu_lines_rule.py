"""Which sweep a launch takes: several lines per wave where there are many, one otherwise.  The choice is by
time alone, so u and J are the same bit for bit either way: lists of few origins (one line per wave) against the same
origins listed often enough for the other, over frequency counts and blocks around its lanes, by rt_solve and
rt_compute_J for static media, by plans (whose padded tables it reads) for moving ones."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

# lengths of the blocks, their widths
BLOCKS = [([1], [0.5]), ([2], [0.5]), ([3], [0.5]), ([5], [0.5]), ([17], [0.5]), ([31], [0.5]), ([63], [0.5]),
          ([64], [0.5]), ([65], [0.5]), ([48, 48], [0.5, 0.5]), ([1, 7, 2, 12], [0.5, 0.5, 0.5, 0.5]),
          ([12, 9], [0.5, 0.6]), ([130], [0.25]), ([259], [0.1]), ([200, 130], [0.1, 0.1]), ([300, 211], [0.1, 0.12])]


def _setup(rt, blocks, moving, fp64):
    import torch
    lens, dx = blocks
    m = synth.tiny_model(500 + sum(lens), P=72, F=sum(lens), moving=moving)
    m.freq = synth.FreqGrid(np.array(lens, np.int32), np.full(len(lens), -2.0), np.array(dx))
    if moving:
        rng = np.random.default_rng(sum(lens))
        m.vel[:] = m.vel * 10.0 ** rng.uniform(-2, 2, (m.P, 1))
    dt = torch.float64 if fp64 else torch.float32
    chi, eta = (torch.as_tensor(x, device="cuda").to(dt) for x in (m.chi, m.eta))
    I_bc = torch.as_tensor(m.I_bc, dtype=torch.float64, device="cuda")
    model = rt.Model.from_numpy(m.pos, m.nbr_off, m.nbr_idx, m.vel)
    few = torch.arange(m.P, dtype=torch.int32, device="cuda")
    # full waves of the one-line sweep in FP32 (64 frequencies) change over at half a million, all others well
    # before 100 000
    F = sum(lens)
    waves = 600_000 if not fp64 and F % 64 in (0, 63) else 110_000
    times = -(-waves // (m.P * 24 * ((F + 63) // 64)))
    return m, model, rt.DirSet.uniform(2), chi, eta, I_bc, few, few.repeat(times), times


@pytest.mark.parametrize("blocks", BLOCKS, ids=lambda b: "+".join(map(str, b[0])))
@pytest.mark.parametrize("fp64", [True, False])
def test_static_lists(rt, blocks, fp64):
    m, model, ds, chi, eta, I_bc, few, many, times = _setup(rt, blocks, False, fp64)
    prec = rt.RT_F64 if fp64 else rt.RT_F32
    args = (m.freq.len, m.freq.dx, I_bc)
    a = rt.solve(model, ds, rt.trace(model, ds, origins=few), chi, eta, *args, origins=few, precision=prec)
    a = a.cpu().numpy()
    for schedule in (rt.SCHED_DIRECT, rt.SCHED_BINNED):
        b = rt.solve(model, ds, rt.trace(model, ds, origins=many), chi, eta, *args, origins=many, precision=prec,
                     schedule=schedule).cpu().numpy()
        assert np.array_equal(b, np.tile(a, (times, 1)))
    c = rt.compute_J(model, ds, chi, eta, *args, origins=many, precision=prec).cpu().numpy()
    assert np.array_equal(c, np.tile(a, (times, 1)))


@pytest.mark.parametrize("blocks", BLOCKS, ids=lambda b: "+".join(map(str, b[0])))
@pytest.mark.parametrize("fp64", [True, False])
def test_moving_plans(rt, blocks, fp64):
    import torch
    m, model, ds, chi, eta, I_bc, few, many, times = _setup(rt, blocks, True, fp64)
    prec = rt.RT_F64 if fp64 else rt.RT_F32
    args = (m.freq.len, m.freq.dx, I_bc)
    a = rt.solve(model, ds, rt.trace(model, ds, origins=few), chi, eta, *args, origins=few, precision=prec)
    a = a.cpu().numpy()
    J = torch.empty((many.numel(), m.F), dtype=chi.dtype, device="cuda")
    plan = rt.Plan(model, ds, chi, eta, *args, J, origins=many, precision=prec, schedule=rt.SCHED_SPATIAL)
    for o in (dict(schedule=rt.SCHED_SPATIAL), dict(schedule=rt.SCHED_BINNED), dict(schedule=rt.SCHED_DIRECT)):
        plan.retune(**o)
        J.zero_()
        plan.run()
        rt.sync_status()
        assert np.array_equal(J.cpu().numpy(), np.tile(a, (times, 1))), o
