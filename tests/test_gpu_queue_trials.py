"""FIFO and SORTED, closed loop, a block per trial (k_queue_run with TRIAL, k_trial_list) against the oracle: membrane trace, spike list,
admission flags, counters, gradients.  One, two, four and eight targets per thread, trials that share spike words, full queues, more
contenders than record slots, synaptic current states, runs of several launches, single steps in between, tapes that end or are too small."""
import numpy as np
import pytest
import torch

from oracle import oracle
from paper_2512_05906_amd import adseq, synth
from tests.helpers import gpu_dropped_set, grad_close, oracle_sets

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,cap", [(adseq.FIFO, 2), (adseq.FIFO, 40), (adseq.SORTED, 5)])
@pytest.mark.parametrize("n,b,fan,d_max,T,rate,syn", [(1, 2, 3, 4, 20, 3000.0, 0), (100, 5, 60, 20, 300, 60.0, 1), (512, 3, 40, 30, 60, 100.0, 0), (513, 2, 90, 25, 80, 100.0, 2),
                                                      (1500, 3, 30, 40, 60, 60.0, 1), (2050, 2, 25, 30, 50, 50.0, 2), (4096, 2, 20, 20, 40, 30.0, 0), (64, 300, 10, 12, 30, 200.0, 0)])
def test_queue_trials(kind, cap, n, b, fan, d_max, T, rate, syn, monkeypatch):
    monkeypatch.setenv("ADSEQ_QUEUE_TRIALS", "1")
    wl = synth.ragged_network(n, fan, d_max, seed=n + b, rate_hz=rate, t=T, b=b, w_mean=0.5 / fan, w_std=0.7 / fan)
    wl.tau_syn_ms, wl.tau_rise_ms = (0.0, 5.0, 5.0)[syn], (0.0, 0.0, 1.0)[syn]
    ref = oracle.Run(wl, kind, cap, n_steps=T, batch=b, log_events=True)
    sim = adseq.Adseq(wl, kind, cap, batch=b, record_tape=True, max_steps=T, tape_spike_capacity=T * b * n, tape_event_capacity=T * b * wl.n_synapses + 1)
    cut = T // 3
    for pieces in ([T], [cut, 1, T - cut - 1]):
        sim.reset()
        n0 = 0
        for p in pieces:
            sim.step(n0) if p == 1 else sim.run(n0, p)
            n0 += p
        torch.cuda.synchronize()
        tape = sim.tape()
        np.testing.assert_array_equal(tape["U"].cpu().numpy().view(np.uint32), ref.U.view(np.uint32))
        raster = ref.spikes.reshape(T, -1) != 0
        off, ids = tape["step_offset"].cpu().numpy(), tape["spike_id"].cpu().numpy()
        np.testing.assert_array_equal(off, np.concatenate([[0], np.cumsum(raster.sum(axis=1))]))
        np.testing.assert_array_equal(ids[:off[-1]], np.concatenate([np.flatnonzero(x) for x in raster]))   # (ascending within a step)
        c, rc = sim.counters(), ref.counters()
        for key in ("enqueued", "dropped", "delivered", "sum_enqueued", "sum_dropped", "sum_delivered"):
            assert c[key] == rc[key], key
        if off[-1] < 3000:
            out = {"step_offset": off, "spike_id": ids, "event_base": tape["event_base"].cpu().numpy()}
            assert gpu_dropped_set(sim, out, wl)[1] == oracle_sets(ref)[1]
        if syn < 2:
            dc = np.random.default_rng(n).normal(0, 1e-3, (b, n)).astype(np.float32)
            gw, gd = ref.backward(dc, None)
            g_w, g_d = torch.empty(wl.n_synapses, device=sim.dev), torch.empty(wl.n_synapses, device=sim.dev)
            sim.backward(torch.from_numpy(dc).to(sim.dev), None, g_w, g_d)
            grad_close(g_w.cpu().numpy(), gw)
            grad_close(g_d.cpu().numpy(), gd)
    sim.close()


def test_tape_ends_and_overflows(monkeypatch):
    """A run past the recorded steps, and one whose spike or event list is too small: counted and reported as by the other kernels."""
    wl = synth.ragged_network(90, 20, 20, seed=4, rate_hz=300.0, t=60, b=3, w_mean=0.02, w_std=0.02)
    ref = oracle.Run(wl, adseq.FIFO, 3, n_steps=60, batch=3)
    for kw in ({"max_steps": 40}, {"max_steps": 60, "tape_spike_capacity": 20}, {"max_steps": 60, "tape_event_capacity": 200}):
        got = []
        for trials in ("0", "1"):
            monkeypatch.setenv("ADSEQ_QUEUE_TRIALS", trials)
            sim = adseq.Adseq(wl, adseq.FIFO, 3, batch=3, record_tape=True, **kw)
            sim.run(0, 60)
            got.append(sim.counters())
            with pytest.raises(Exception):
                sim.backward(torch.zeros(270, device=sim.dev), None, torch.empty(wl.n_synapses, device=sim.dev), torch.empty(wl.n_synapses, device=sim.dev))
            sim.close()
        assert got[0] == got[1]
        for key in ("enqueued", "dropped", "delivered"):
            assert got[1][key] == ref.counters()[key]


@pytest.mark.parametrize("kind,cap", [(adseq.FIFO, 3), (adseq.SORTED, 5)])
def test_short_calls_between_long_ones(kind, cap):
    """Calls of a few steps go by blocks over the whole chip, longer ones by a block per trial: queues, tape and counters pass from one to the other."""
    n, b, pieces = 90, 3, (40, 5, 12, 4, 4, 30, 1, 6, 8)
    T = sum(pieces)
    wl = synth.ragged_network(n, 25, 20, seed=9, rate_hz=300.0, t=T, b=b, w_mean=0.02, w_std=0.02)
    ref = oracle.Run(wl, kind, cap, n_steps=T, batch=b)
    sim = adseq.Adseq(wl, kind, cap, batch=b, record_tape=True, max_steps=T, tape_spike_capacity=T * b * n, tape_event_capacity=T * b * wl.n_synapses + 1)
    from torch.profiler import ProfilerActivity, profile
    ran, at = [], 0
    for p in pieces:
        with profile(activities=[ProfilerActivity.CUDA]) as prof:
            sim.run(at, p)
            torch.cuda.synchronize()
        ran.append("k_trial_list" in " ".join(e.name for e in prof.events()))
        at += p
    assert ran == [p >= 8 for p in pieces]                 # (the last step of a call goes by itself)
    assert np.array_equal(sim.tape()["U"].cpu().numpy().reshape(-1).view(np.uint32), ref.U.reshape(-1).view(np.uint32))
    c, rc = sim.counters(), ref.counters()
    for key in ("enqueued", "dropped", "delivered", "sum_enqueued", "sum_dropped", "sum_delivered"):
        assert c[key] == rc[key], key
    dc = np.random.default_rng(n).normal(0, 1e-3, (b, n)).astype(np.float32)
    gw, gd = ref.backward(dc, None)
    g_w, g_d = torch.empty(wl.n_synapses, device=sim.dev), torch.empty(wl.n_synapses, device=sim.dev)
    sim.backward(torch.from_numpy(dc).to(sim.dev), None, g_w, g_d)
    np.testing.assert_allclose(g_w.cpu().numpy(), gw, rtol=1e-5, atol=1e-6)
    np.testing.assert_allclose(g_d.cpu().numpy(), gd, rtol=1e-5, atol=1e-6)
    sim.close()
