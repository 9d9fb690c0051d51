"""The wavefront autotuner on a register plan that has a one-wavefront form for
large batches: the cut is timed as the cut, and the form is not lost.

A batch of 400 bitstrings x 1024 slices of 6x6x25 takes about 0.2 ms on the
form and 0.6 ms on the four-wavefront cut.  The bounds, 1.4 times the untuned
call and 0.7 times the cut, lie between the two."""
import pytest

import paper_1805_01450_amd as q
from workload import generate_circuit, random_bitstrings

pytestmark = pytest.mark.gpu
N_BS = 400


def _ms(p, bits):
    """One run, the best of five groups of five."""
    import torch
    d_bits = torch.from_numpy(bits).cuda()
    out = torch.empty((len(bits), 4), dtype=torch.float64, device="cuda")
    ws = p.workspace(len(bits))
    e0, e1 = (torch.cuda.Event(enable_timing=True) for _ in range(2))
    best = float("inf")
    for group in range(6):
        e0.record()
        for _ in range(5):
            q.qgm_amplitudes_device(p.h, d_bits, None, 0, 1 << p.k, ws, out)
        e1.record()
        torch.cuda.synchronize()
        if group:
            best = min(best, e0.elapsed_time(e1) / 5)
    return best


@pytest.fixture(scope="module")
def made():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    c = q.Circuit(generate_circuit(6, 25, 0))
    sl, order = c.plan_slices(k_req=10, time_budget_s=1.0, flags=q.QGM_PLAN_DETERMINISTIC)
    bits = random_bitstrings(36, N_BS, 21)
    p = q.Plan(c, sl, order, prec=q.QGM_C64)
    cut = q.Plan(c, sl, order, prec=q.QGM_C64, waves=p.stats()["waves"])  # has no such form
    assert p.stats()["waves"] > 1
    ms, cut_ms = _ms(p, bits), _ms(cut, bits)
    print("[tune] untuned", ms, "cut", cut_ms, flush=True)
    assert ms <= 0.7 * cut_ms  # the form runs
    return c, sl, order, bits, p.amplitudes(bits), ms


@pytest.mark.parametrize("tuned_for,waves", [(N_BS, 1), (1, None)])
def test_tuning_keeps_the_form(made, tuned_for, waves):
    c, sl, order, bits, want, ms = made
    p = q.Plan(c, sl, order, prec=q.QGM_C64)
    chosen = p.autotune(tuned_for)
    got_ms = _ms(p, bits)
    print("[tune] for", tuned_for, "chose", chosen, got_ms, flush=True)
    if chosen in (1, p.stats()["waves"]):  # its own cut or the form: both kept
        assert got_ms <= 1.4 * ms
        assert (p.amplitudes(bits) == want).all()
        assert (p.amplitudes(bits[:1]) == want[:1]).all()
    assert waves is None or chosen == waves
