"""The row layouts that only models of gigabytes of rows take, forced on small ones: 64-bit row offsets, and
row codes without the rows' lengths.  Lists are the oracle's bit for bit, on irregular points, on rows long
enough that their length is kept in the row, and on a lattice (steps that the FP64 rule decides)."""
import ctypes as C

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

CREATE = "_ZN2rt12model_createEPKdlPKlPKilPKfS5_bP12ihipStream_tPP8rt_modeli"  # rt::model_create


def _model(rt, m, layout):
    gm = rt.Model.from_numpy(m.pos, m.nbr_off, m.nbr_idx, None)
    fn = C.CDLL(rt.binding.LIB_PATH)[CREATE]
    fn.restype = C.c_int32
    fn.argtypes = [C.c_void_p, C.c_int64, C.c_void_p, C.c_void_p, C.c_int64, C.c_void_p, C.c_void_p, C.c_bool,
                   C.c_void_p, C.c_void_p, C.c_int32]
    h = C.c_void_p()
    assert fn(gm.pos.data_ptr(), m.P, gm.nbr_off.data_ptr(), gm.nbr_idx.data_ptr(), gm.nbr_idx.numel(), None, None,
              True, None, C.byref(h), layout) == 0
    rt.load().rt_model_destroy(gm._h)
    gm._h = h
    return gm


def _full(P):
    m = synth.tiny_model(95, P=max(P, 40))
    a, b = np.triu_indices(P, 1)
    off, idx = synth.models.csr_from_edges(P, a, b)
    pos = np.random.default_rng(P).normal(size=(P, 3))
    return synth.Model("full", pos, off, idx, None, m.chi[:1].repeat(P, 0), m.eta[:1].repeat(P, 0), m.freq, m.I_bc)


@pytest.mark.parametrize("layout", [1, 2], ids=["far", "wide"])
@pytest.mark.parametrize("name", ["tiny", "rows of 56", "rows of 57", "rows of 99", "lattice"])
def test_forced_layouts(rt, orc, name, layout):
    import torch
    m = (synth.tiny_model(96, P=90) if name == "tiny" else synth.lattice_model(5) if name == "lattice"
         else _full(int(name.split()[-1]) + 1))
    model = _model(rt, m, layout)
    ds = rt.DirSet.uniform(2)
    _, dirs, _ = orc.dirset_uniform(2)
    origins = np.arange(0, m.P, 2, dtype=np.int32)
    org = torch.as_tensor(origins, device="cuda")
    e = orc.trace_all(m, dirs, origins)
    chi, eta, I_bc = (torch.as_tensor(x, dtype=torch.float64, device="cuda") for x in (m.chi, m.eta, m.I_bc))
    J = torch.empty((len(origins), m.F), dtype=torch.float64, device="cuda")
    plan = rt.Plan(model, ds, chi, eta, m.freq.len, m.freq.dx, I_bc, J, origins=org, precision=rt.RT_F64,
                   trace_lanes=8)
    plan.run()
    rt.sync_status()
    for g in (plan.rays(), rt.trace(model, ds, origins=org)):
        got = [x.cpu().numpy() for x in g]
        assert np.array_equal(got[0], e[0])
        assert np.array_equal(got[1], e[1])
        assert np.array_equal(got[2].view(np.uint64), e[2].view(np.uint64))
