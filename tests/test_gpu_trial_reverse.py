"""Reverse sweep of small networks in one launch, a workgroup per trial (k_bwd_trial), against the oracle: both gradients, gradient modes,
cotangents, queue kinds; rows of a run in LDS as a whole and in pieces, sizes around a wavefront and the largest, trials that share
spike words (with rows of another trial's spikes in front), empty rows, rows of more than 64 and 256 entries, steps with more pieces than
are requested ahead and than the list holds, runs shorter than what is loaded ahead."""
import numpy as np
import pytest
import torch

from oracle import oracle
from paper_2512_05906_amd import adseq, synth
from tests.helpers import grad_close

pytestmark = pytest.mark.gpu

CASES = [  # n, b, fan, d_max, T, rate, tau_syn
    (1, 1, 3, 4, 12, 3000.0, 0.0), (63, 3, 20, 30, 60, 300.0, 0.0), (64, 2, 150, 7, 50, 200.0, 5.0), (65, 4, 10, 250, 300, 150.0, 0.0),
    (100, 1, 300, 60, 90, 900.0, 0.0), (513, 2, 40, 200, 230, 60.0, 5.0), (1000, 3, 60, 50, 70, 100.0, 0.0), (1024, 1, 30, 120, 140, 3000.0, 0.0),
    (1023, 2, 700, 45, 40, 40.0, 0.0), (200, 2, 12, 9, 3, 2000.0, 0.0)]


@pytest.mark.parametrize("kind,cap", [(adseq.RING, 0), (adseq.FIFO, 3), (adseq.SORTED, 20), (adseq.SYN_LATEST, 1)])
@pytest.mark.parametrize("n,b,fan,d_max,T,rate,tau_syn", CASES)
def test_trial_reverse(kind, cap, n, b, fan, d_max, T, rate, tau_syn, monkeypatch):
    monkeypatch.setenv("ADSEQ_REVERSE_TRIALS", "1")     # whatever spikes
    wl = synth.ragged_network(n, fan, d_max, seed=n + b, rate_hz=rate, t=T, b=b, w_mean=0.4 / fan, w_std=0.5 / fan)
    wl.tau_syn_ms = tau_syn
    rng = np.random.default_rng(n)
    for mode, du in ((adseq.SURR_SUPERSPIKE, False), (adseq.GRAD_SPIKE_TIME, True)):
        ref = oracle.Run(wl, kind, cap, n_steps=T, batch=b, surrogate=mode)
        sim = adseq.Adseq(wl, kind, cap, batch=b, record_tape=True, max_steps=T, surrogate=mode, tape_spike_capacity=T * b * n + 64,
                          tape_event_capacity=(T * b + 1) * wl.n_synapses + 64)
        sim.run(0, T)
        dc = None if du else rng.normal(0, 1e-2, (b, n)).astype(np.float32)
        dU = rng.normal(0, 1e-2, (T, b, n)).astype(np.float32) if du else None
        gw, gd = ref.backward(dc, dU)
        g_w, g_d = torch.empty(wl.n_synapses, device=sim.dev), torch.empty(wl.n_synapses, device=sim.dev)
        for _ in range(2):
            sim.backward(None if dc is None else torch.from_numpy(dc).to(sim.dev), None if dU is None else torch.from_numpy(dU).to(sim.dev), g_w, g_d)
            # (an element may be what is left of terms as large as the largest gradient: fp32 sums of them in another order differ by some
            # eight roundings, 8 x 6e-8 of it, which the absolute part has to allow beyond 1e-6)
            for got, want in ((g_w, gw), (g_d, gd)):
                grad_close(got.cpu().numpy(), want, atol=1e-6 + 5e-7 * float(np.abs(want).max(initial=0.0)))
        sim.close()


@pytest.mark.parametrize("kind,cap", [(adseq.RING, 0), (adseq.FIFO, 3)])
@pytest.mark.parametrize("n,d_max,rate", [(64, 20, 150.0), (300, 30, 200.0), (200, 15, 20000.0)])
def test_steps_that_hand_out_nothing(kind, cap, n, d_max, rate, monkeypatch):
    """Steps whose only spikes are of neurons without synapses, which the spike-time rule takes through the membrane value of the step before
    nonetheless, between steps with rows."""
    monkeypatch.setenv("ADSEQ_REVERSE_TRIALS", "1")
    T, b = 150, 3
    wl = synth.ragged_network(n, 12, d_max, seed=n, rate_hz=rate, t=T, b=b, w_mean=0.05, w_std=0.05)
    keep = np.repeat(np.arange(n) % 4 == 0, np.diff(wl.row_ptr))
    wl.row_ptr = np.concatenate([[0], np.cumsum(np.where(np.arange(n) % 4 == 0, np.diff(wl.row_ptr), 0))]).astype(np.int64)
    wl.col, wl.weight, wl.delay_steps = wl.col[keep], wl.weight[keep], wl.delay_steps[keep]
    ref = oracle.Run(wl, kind, cap, n_steps=T, batch=b, surrogate=adseq.GRAD_SPIKE_TIME)
    per_step = ref.spikes.reshape(T, b, n).sum(axis=2)
    with_rows = (ref.spikes.reshape(T, b, n) * (np.diff(wl.row_ptr) > 0)).sum(axis=2)
    assert rate > 1000.0 or ((per_step > 0) & (with_rows == 0)).sum() > 5
    dU = np.random.default_rng(n).normal(0, 1e-2, (T, b, n)).astype(np.float32)
    gw, gd = ref.backward(None, dU)
    sim = adseq.Adseq(wl, kind, cap, batch=b, record_tape=True, max_steps=T, surrogate=adseq.GRAD_SPIKE_TIME, tape_spike_capacity=T * b * n + 64)
    sim.run(0, T)
    g_w, g_d = torch.empty(wl.n_synapses, device=sim.dev), torch.empty(wl.n_synapses, device=sim.dev)
    sim.backward(None, torch.from_numpy(dU).to(sim.dev), g_w, g_d)
    for got, want in ((g_w, gw), (g_d, gd)):   # (bound of the absolute part: see above)
        grad_close(got.cpu().numpy(), want, atol=1e-6 + 5e-7 * float(np.abs(want).max(initial=0.0)))
    sim.close()


def _kernels(call):
    from torch.profiler import ProfilerActivity, profile
    with profile(activities=[ProfilerActivity.CUDA]) as p:
        call()
        torch.cuda.synchronize()
    return " ".join(e.name for e in p.events())


@pytest.mark.parametrize("rate,trials", [(20.0, True), (3000.0, False)])
def test_the_line_is_on_the_spikes(rate, trials):
    """Few spikes: a workgroup per trial; many: the kernels over the whole chip."""
    n, T = 900, 80
    wl = synth.ragged_network(n, 60, 50, seed=3, rate_hz=rate, t=T, b=8, w_mean=0.001, w_std=0.001)
    sim = adseq.Adseq(wl, adseq.RING, 0, batch=8, record_tape=True, max_steps=T)
    sim.run(0, T)
    g_w, g_d = torch.empty(wl.n_synapses, device=sim.dev), torch.empty(wl.n_synapses, device=sim.dev)
    names = _kernels(lambda: sim.backward(torch.ones(8 * n, device=sim.dev), None, g_w, g_d))
    assert ("k_bwd_trial" in names) == trials and ("k_bwd_flow" in names) != trials
    sim.close()


@pytest.mark.parametrize("b", [54, 109])
@pytest.mark.parametrize("of_the_line,trials", [(0.93, True), (1.07, False)])
def test_all_spikes_are_counted_for_the_line(b, of_the_line, trials):
    """Spikes a little below and a little above the line (7 pieces of work per step and trial), summed by one block and by several, cells
    that no 4 divides: a share of the cells left out or taken twice would turn the choice."""
    n, T = 301, 40
    wl = synth.ragged_network(n, 60, 50, seed=3, rate_hz=1.0, t=T, b=b, w_mean=1e-4, w_std=1e-5)
    wl.ext_weight = 1.5                                    # (every event of the drive is a spike)
    line = 7.0 / (1.0 + wl.n_synapses / n / 64.0)          # spikes per step and trial
    wl.ext_rate_hz = of_the_line * line / n * 1e4
    sim = adseq.Adseq(wl, adseq.RING, 0, batch=b, record_tape=True, max_steps=T)
    sim.run(0, T)
    counts = torch.empty(b * n, dtype=torch.int32, device=sim.dev)
    sim.spike_counts(counts)
    assert abs(int(counts.sum()) / (T * b) / line - of_the_line) < 0.05
    g_w, g_d = torch.empty(wl.n_synapses, device=sim.dev), torch.empty(wl.n_synapses, device=sim.dev)
    names = _kernels(lambda: sim.backward(torch.ones(b * n, device=sim.dev), None, g_w, g_d))
    assert ("k_bwd_trial" in names) == trials and ("k_bwd_flow" in names) != trials
    sim.close()
