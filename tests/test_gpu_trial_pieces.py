"""Small ring networks whose delay line does not fit LDS: a run in one launch with a spike's row in two to four pieces (k_trial_run with
PIECES) against the oracle: trace, counters, gradients; runs cut anywhere -- in and between windows, within the delays of held spikes --,
with single steps and a current from outside in between, so that the window and the spike words that a launch leaves are read by the other
kernels and the other way round; delays of exactly one and two pieces, rows of more than 64 and 256 entries per piece, shared spike words."""
import numpy as np
import pytest
import torch

from oracle import oracle
from paper_2512_05906_amd import adseq, synth
from tests.helpers import grad_close

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,b,fan,d_max,T,rate,tau_syn,tau_rise,continuous", [
    (1000, 2, 60, 50, 400, 60.0, 0.0, 0.0, False), (1024, 1, 30, 45, 420, 2500.0, 0.0, 0.0, False), (1021, 3, 40, 62, 330, 200.0, 5.0, 0.0, True),
    (600, 2, 50, 200, 500, 80.0, 5.0, 1.0, False), (700, 1, 1100, 60, 300, 30.0, 0.0, 0.0, False), (900, 2, 80, 100, 380, 100.0, 0.0, 0.0, False)])
def test_trial_pieces(n, b, fan, d_max, T, rate, tau_syn, tau_rise, continuous, monkeypatch):
    monkeypatch.setenv("ADSEQ_RING_TRIALS", "1")
    wl = synth.ragged_network(n, fan, d_max, seed=n, rate_hz=rate, t=T, b=b, w_mean=0.6 / fan, w_std=0.6 / fan, continuous=continuous)
    wl.tau_syn_ms, wl.tau_rise_ms = tau_syn, tau_rise
    ext = np.zeros((T, b, n), np.float32)
    ext[150:153] = (np.random.default_rng(1).random((3, b, n)) < 0.1) * 1.2
    ref = oracle.Run(wl, oracle.RING, 0, n_steps=T, batch=b, i_ext=ext, n_threads=8)
    sim = adseq.Adseq(wl, adseq.RING, 0, batch=b, record_tape=True, max_steps=T)
    cur = torch.from_numpy(ext).to(sim.dev)
    for first in ((150,), (64, 86), (67, 1, 82)):     # then three single steps with the current, then two launches
        sim.reset()
        s = 0
        for p in first:
            sim.step(s) if p == 1 else sim.run(s, p)
            s += p
        for s in range(150, 153):
            sim.step(s, cur[s])
        sim.run(153, 75)
        sim.run(228, T - 228)
        torch.cuda.synchronize()
        np.testing.assert_array_equal(sim.tape()["U"].cpu().numpy().view(np.uint32), ref.U.view(np.uint32))
        c, rc = sim.counters(), ref.counters()
        for key in ("enqueued", "dropped", "delivered", "sum_enqueued", "sum_dropped", "sum_delivered"):
            assert c[key] == rc[key], key
    if tau_rise == 0.0:
        dc = np.random.default_rng(n).normal(0, 1e-3, (b, n)).astype(np.float32)
        gw, gd = ref.backward(dc, None)
        g_w, g_d = torch.empty(wl.n_synapses, device=sim.dev), torch.empty(wl.n_synapses, device=sim.dev)
        sim.backward(torch.from_numpy(dc).to(sim.dev), None, g_w, g_d)
        for got, want in ((g_w, gw), (g_d, gd)):   # (bound of the absolute part: see test_gpu_trial_reverse.py)
            grad_close(got.cpu().numpy(), want, atol=1e-6 + 5e-7 * float(np.abs(want).max(initial=0.0)))
    sim.close()


@pytest.mark.parametrize("b,least", [(1, 128), (16, 64)])
def test_calls_that_are_too_short(b, least):
    """At the default line calls below the least number of steps go by the other kernels, and each takes over from the other."""
    n, d_max, pieces = 1000, 50, (least - 1, least, 3, least + 5)
    T = sum(pieces)
    wl = synth.ragged_network(n, 200, d_max, seed=b, rate_hz=40.0, t=T, b=b, w_mean=0.004, w_std=0.004)
    ref = oracle.Run(wl, oracle.RING, 0, n_steps=T, batch=b, n_threads=8)
    sim = adseq.Adseq(wl, adseq.RING, 0, batch=b, record_tape=True, max_steps=T)
    from torch.profiler import ProfilerActivity, profile
    ran, at = [], 0
    for p in pieces:
        with profile(activities=[ProfilerActivity.CUDA]) as prof:
            sim.run(at, p)
            torch.cuda.synchronize()
        ran.append("k_trial_run" in " ".join(e.name for e in prof.events()))
        at += p
    assert ran == [p >= least for p in pieces]
    np.testing.assert_array_equal(sim.tape()["U"].cpu().numpy().view(np.uint32), ref.U.view(np.uint32))
    c, rc = sim.counters(), ref.counters()
    for key in ("enqueued", "dropped", "delivered", "sum_enqueued", "sum_dropped", "sum_delivered"):
        assert c[key] == rc[key], key
    sim.close()


def test_short_calls_under_capture():
    """A captured call of 64 steps and more is recorded as the kernel whose workgroups wait for nobody; its replays leave what eager calls leave."""
    n, T = 1000, 70
    wl = synth.ragged_network(n, 200, 50, seed=2, rate_hz=60.0, t=T, b=1, w_mean=0.004, w_std=0.004)
    ref = oracle.Run(wl, oracle.RING, 0, n_steps=T, batch=1, n_threads=8)
    sim = adseq.Adseq(wl, adseq.RING, 0, batch=1, record_tape=True, max_steps=T)
    sim.reset(); sim.run(0, T)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        sim.reset()
        sim.run(0, T)
    U = sim.membrane_tape(T)
    from torch.profiler import ProfilerActivity, profile
    for _ in range(3):
        U.zero_()
        with profile(activities=[ProfilerActivity.CUDA]) as prof:
            graph.replay()
            torch.cuda.synchronize()
        names = " ".join(e.name for e in prof.events())
        assert "k_trial_run" in names and "k_fwd_chip" not in names and "k_run_xcd" not in names
        np.testing.assert_array_equal(U.cpu().numpy().view(np.uint32), ref.U.view(np.uint32).reshape(U.shape))
    sim.close()
