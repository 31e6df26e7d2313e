"""A plan that holds padded copies of its tables gives them up when an option needs the memory: changing
to the binned schedule with less memory free than its item list takes still works, and J stays the same."""
import pytest

import synth

pytestmark = pytest.mark.gpu

MB = 1 << 20


def test_retune_when_memory_is_short(rt):
    """50 000 points, 2048 frequencies, 96 pairs: copies of 822 MB, an item list of 614 MB; 400 MB left free."""
    import torch
    m = synth.wind_model(P=50_000, F=8)
    F = 2048
    model = rt.Model.from_numpy(m.pos, m.nbr_off, m.nbr_idx, m.vel)
    rho = torch.as_tensor(m.chi[:, :1], dtype=torch.float32, device="cuda")
    chi = rho * torch.linspace(0.5, 1.5, F, device="cuda")[None, :]
    eta = 0.5 * chi
    I_bc = torch.zeros(F, dtype=torch.float64, device="cuda")
    J = torch.empty((m.P, F), dtype=torch.float32, device="cuda")
    ds = rt.DirSet.uniform(4)
    rt.release_cached_memory()
    plan = rt.Plan(model, ds, chi, eta, [F], [0.01], I_bc, J, schedule=rt.SCHED_SPATIAL)
    plan.run()
    rt.sync_status()
    before = J.clone()
    torch.cuda.empty_cache()
    filler = []
    try:
        for _ in range(10):  # memory that was freed just before may be counted late
            free = torch.cuda.mem_get_info()[0]
            if free < 500 * MB:
                break
            filler.append(torch.empty(free - 400 * MB, dtype=torch.uint8, device="cuda"))
        assert 300 * MB < torch.cuda.mem_get_info()[0] < 600 * MB
        plan.retune(schedule=rt.SCHED_BINNED)
        J.zero_()
        plan.run()
        rt.sync_status()
        assert torch.equal(J, before)
    finally:
        del filler, plan
        torch.cuda.empty_cache()
        rt.release_cached_memory()
