"""The walk's FP32 filter and row layout where they can go wrong: every list equals the
oracle's FP64 rule bit for bit on meshes whose scale, offset or regularity leaves the
filter little room, and on rows of every length around the fours and passes they are
read in."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


def _check(rt, orc, m, nside, origins, lanes=(0,)):
    import torch
    model = rt.Model.from_numpy(m.pos, m.nbr_off, m.nbr_idx, m.vel)
    ds = rt.DirSet.uniform(nside)
    org = torch.as_tensor(origins.astype(np.int32), device="cuda")
    _, dirs, _ = orc.dirset_uniform(nside)
    e = orc.trace_all(m, dirs, origins.astype(np.int32))
    got = [rt.trace(model, ds, origins=org)]
    chi = torch.as_tensor(m.chi, device="cuda")
    eta = torch.as_tensor(m.eta, device="cuda")
    I_bc = torch.as_tensor(m.I_bc, device="cuda")
    J = torch.empty((len(origins), m.F), dtype=torch.float64, device="cuda")
    for gl in lanes:
        plan = rt.Plan(model, ds, chi, eta, m.freq.len, m.freq.dx, I_bc, J, origins=org, precision=rt.RT_F64,
                       schedule=rt.SCHED_SPATIAL, trace_lanes=gl)
        plan.run()
        rt.sync_status()
        got.append(plan.rays())
        del plan
    for g in got:
        off, ids, Z = (x.cpu().numpy() for x in g)
        assert np.array_equal(off, e[0])
        assert np.array_equal(ids, e[1])
        assert np.array_equal(Z.view(np.uint64), e[2].view(np.uint64))


def _with_pos(m, pos):
    return synth.Model(m.name, np.ascontiguousarray(pos), m.nbr_off, m.nbr_idx, m.vel, m.chi, m.eta, m.freq, m.I_bc)


@pytest.mark.parametrize("scale", [1e-300, 1e-160, 1e-30, 3.0, 1e30, 1e145])
def test_scaled_meshes(rt, orc, scale):
    m = synth.tiny_model(91, P=90)
    _check(rt, orc, _with_pos(m, m.pos * scale), 2, np.arange(m.P))


@pytest.mark.parametrize("far", [1e3, 1e8, 1e12, 1e15])
def test_offset_meshes(rt, orc, far):
    """Coordinates whose differences keep ever fewer digits: equal and zero edges at the end."""
    m = synth.tiny_model(92, P=90)
    _check(rt, orc, _with_pos(m, m.pos + far * np.array([1.0, -0.5, 0.25])), 2, np.arange(m.P))


@pytest.mark.parametrize("squeeze", [1e-4, 1e-9, 1e-20, 0.0])
def test_flat_meshes(rt, orc, squeeze):
    """One axis far thinner than the others (0: all points in a plane, many exact ties)."""
    m = synth.tiny_model(93, P=90)
    _check(rt, orc, _with_pos(m, m.pos * np.array([1.0, 1.0, squeeze])), 2, np.arange(m.P))


def test_mixed_edge_lengths(rt, orc):
    """Clusters of edge 1e-9 joined by edges of order one."""
    rng = np.random.default_rng(94)
    m = synth.tiny_model(94, P=80)
    pos = rng.uniform(-1, 1, (20, 3))[np.arange(m.P) % 20] + 1e-9 * rng.normal(size=(m.P, 3))
    _check(rt, orc, _with_pos(m, pos), 2, np.arange(m.P))


def test_lattice_all_lanes(rt, orc):
    m = synth.lattice_model(6)
    _check(rt, orc, m, 2, np.arange(m.P), lanes=(4, 8, 16))


@pytest.mark.parametrize("P", [5, 24, 25, 26, 61, 62, 70, 300])
def test_long_rows(rt, orc, P):
    """Every point a neighbour of every other: rows of P - 1 records (a fours count that
    saturates its four bits at 15, i.e. from 57 records on)."""
    rng = np.random.default_rng(P)
    m = synth.tiny_model(95, P=max(P, 40))
    pos = rng.normal(size=(P, 3))
    a, b = np.triu_indices(P, 1)
    off, idx = synth.models.csr_from_edges(P, a, b)
    full = synth.Model("full", pos, off, idx, None, m.chi[:1].repeat(P, 0), m.eta[:1].repeat(P, 0), m.freq, m.I_bc)
    _check(rt, orc, full, 1, np.arange(min(P, 70)), lanes=(4, 8, 16))
