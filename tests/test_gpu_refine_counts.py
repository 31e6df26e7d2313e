"""The refined sweeps' kernels (velocity sampling alone, optical depth alone, both) at split counts
around the 64 sub-points that a wave forms at once, against the oracle: FP64 within 1e-12 and FP32
within 1e-4 relative, as for every refined line."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cap", [63, 64, 65, 66, 128, 129, 130, 1024])
@pytest.mark.parametrize("dv_max,dtau_max", [(0.01, 0.0), (0.0, 0.005), (0.02, 0.5)])
def test_split_counts(rt, orc, cap, dv_max, dtau_max):
    import torch
    m = synth.tiny_model(640, P=40, F=10, moving=True)  # velocity steps of 3 Doppler widths: 300 parts and more
    c32, e32, c64, e64 = synth.to_fp32_tables(m.chi, m.eta)
    model, ds = rt.Model.from_numpy(m.pos, m.nbr_off, m.nbr_idx, m.vel), rt.DirSet.uniform(1)
    _, dirs, w2 = orc.dirset_uniform(1)
    org = torch.arange(m.P, dtype=torch.int32, device="cuda")
    rays = rt.trace(model, ds, origins=org)
    kw = dict(dv_max=dv_max, dtau_max=dtau_max)
    Je = orc.compute_J(m, dirs, w2, chi=c64, eta=e64, max_sub=cap, **kw)
    I_bc = torch.as_tensor(m.I_bc, dtype=torch.float64, device="cuda")
    for prec, chi, eta, tol in ((rt.RT_F64, c64, e64, 1e-12), (rt.RT_F32, c32, e32, 1e-4)):
        J = rt.solve(model, ds, rays, torch.as_tensor(chi, device="cuda"), torch.as_tensor(eta, device="cuda"),
                     m.freq.len, m.freq.dx, I_bc, origins=org, precision=prec, max_substeps=cap, **kw).cpu().numpy()
        assert np.max(np.abs(J - Je) / np.abs(Je)) <= tol
