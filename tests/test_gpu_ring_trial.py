"""Small ring networks, closed loop, a run in one launch with a workgroup per trial (k_trial_run) against the oracle: trace bit for
bit, counters, gradients; one wavefront and many, trials that share a spike word, rows whose front does not fit LDS, runs cut
into pieces and mixed with single steps and with the queue entry points in the middle of a window."""
import numpy as np
import pytest
import torch

from oracle import oracle
from paper_2512_05906_amd import adseq, synth
from tests import helpers as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,b,T,d_max,fan,rate,gain,tau_syn,tau_rise,continuous", [
    (63, 1, 300, 130, 40, 900.0, 1.0, 0.0, 0.0, False), (100, 3, 130, 1, 60, 900.0, 0.6, 0.0, 0.0, False),
    (1000, 3, 160, 30, 100, 400.0, 0.6, 0.0, 0.0, False), (903, 2, 130, 35, 90, 400.0, 0.6, 5.0, 0.0, True),
    (1024, 2, 100, 31, 50, 400.0, 0.6, 5.0, 1.0, False), (150, 2, 90, 5, 1500, 900.0, 0.6, 0.0, 0.0, False),
    (200, 7, 140, 3, 30, 2500.0, 1.5, 0.0, 0.0, False), (1000, 2, 80, 20, 524, 2500.0, 0.3, 0.0, 0.0, False),
    (256, 3, 90, 40, 1300, 3000.0, 0.3, 5.0, 0.0, True), (100, 2, 90, 60, 1300, 3000.0, 0.3, 0.0, 0.0, False)])
def test_ring_trial(n, b, T, d_max, fan, rate, gain, tau_syn, tau_rise, continuous, monkeypatch):
    wl = synth.ragged_network(n, fan, d_max, seed=n, rate_hz=rate, t=T, b=b, w_mean=gain / fan, w_std=gain / fan, continuous=continuous)
    wl.tau_syn_ms, wl.tau_rise_ms = tau_syn, tau_rise
    words = (d_max + 1) * ((n + 63) // 64) + ((d_max + 1) * n + 1) // 2 + n
    assert wl.n_synapses <= 262144 and words <= 18432   # (the kernel takes it)
    ref = oracle.Run(wl, adseq.RING, 0, n_steps=T, batch=b, n_threads=8)
    assert ref.spikes.sum() > 50
    rc = ref.counters()
    dc = np.random.default_rng(n).normal(0, 1e-3, (b, n)).astype(np.float32)
    gw, gd = ref.backward(dc, None)
    for trials, pieces, record in (("1", [T], True), ("1", [65, T - 65], True), ("1", [T - 9, "s", 8], True), ("1", [T - 19, 16, 3], False),
                                   ("0", [T], True)):
        monkeypatch.setenv("ADSEQ_RING_TRIALS", trials)
        sim = adseq.Adseq(wl, adseq.RING, 0, batch=b, record_tape=record, max_steps=T)
        for _ in range(2):   # (the second time after a reset)
            sim.reset()
            k = 0
            for p in pieces:
                if p == "s":
                    sim.step(k); k += 1
                else:
                    sim.run(k, p); k += p
            for _ in range(2):   # (asking for the counters changes nothing)
                c = sim.counters()
                for key in ("enqueued", "dropped", "delivered", "sum_enqueued", "sum_dropped", "sum_delivered"):
                    assert c[key] == rc[key], (key, trials, pieces)
                assert c["error_bits"] & ~64 == 0 and c["tape_spikes"] == ref.spikes.sum()
        if record:
            np.testing.assert_array_equal(sim.tape()["U"].cpu().numpy().view(np.uint32), ref.U.view(np.uint32))
            cnt = torch.empty(b * n, dtype=torch.int32, device=sim.dev)
            sim.spike_counts(cnt)
            np.testing.assert_array_equal(cnt.cpu().numpy().reshape(b, -1), ref.spikes.sum(axis=0))
            g_w, g_d = (torch.empty(wl.n_synapses, device=sim.dev) for _ in range(2))
            sim.backward(torch.from_numpy(dc).to(sim.dev), None, g_w, g_d)
            torch.cuda.synchronize()
            H.grad_close(g_w.cpu().numpy(), gw)
            H.grad_close(g_d.cpu().numpy(), gd)
        sim.close()


@pytest.mark.parametrize("n,b", [(100, 16), (250, 8), (1000, 1)])
@pytest.mark.parametrize("record", [True, False])
def test_ring_trial_is_what_runs(n, b, record, monkeypatch):
    """Every block size is reached: with one poll per wait the other forward kernels' waits run out, and a workgroup per trial has none;
    calls shorter than 64 steps go by the others."""
    monkeypatch.setenv("ADSEQ_RING_RESIDENT_SPINS", "1")
    wl = synth.ragged_network(n, 40, 20, seed=4, rate_hz=400.0, t=64, b=b, w_mean=0.01, w_std=0.01)
    for trials, steps in (("1", 64), ("0", 64), ("1", 63)):
        monkeypatch.setenv("ADSEQ_RING_TRIALS", trials)
        sim = adseq.Adseq(wl, adseq.RING, 0, batch=b, record_tape=record, max_steps=64)
        sim.run(0, steps)
        assert (sim.counters()["error_bits"] & 32 == 0) == (trials == "1" and steps == 64)
        sim.close()


@pytest.mark.parametrize("T", [96, 107, 150])
def test_ring_trial_then_queue_entry_points(T, monkeypatch):
    """What is in flight after a run is delivered step by step as after the other kernels, at a window's first step and inside one, and
    so are the events of spikes listed on top of it; the steps beyond the tape are run too."""
    b, n = 2, 120
    wl = synth.ragged_network(n, 40, 60, seed=9, rate_hz=900.0, t=T, b=b, w_mean=0.02, w_std=0.02)
    got = []
    for trials in ("1", "0"):
        monkeypatch.setenv("ADSEQ_RING_TRIALS", trials)
        sim = adseq.Adseq(wl, adseq.RING, 0, batch=b, record_tape=True, max_steps=T - 20)
        sim.run(0, T)
        cur = torch.zeros((70, b * n), device=sim.dev)
        ids = torch.arange(0, b * n, 3, dtype=torch.int32, device=sim.dev)
        count = torch.tensor([ids.numel()], dtype=torch.int32, device=sim.dev)
        for k in range(70):
            sim.deliver(T + k, cur[k])
            if k in (0, 5, 9):
                sim.enqueue(T + k, ids, count)
        got.append((cur.cpu().numpy(), sim.counters()))
        sim.close()
    np.testing.assert_array_equal(got[0][0], got[1][0])
    assert np.abs(got[0][0]).sum() > 0
    for key in ("enqueued", "dropped", "delivered", "sum_enqueued", "sum_dropped", "sum_delivered"):
        assert got[0][1][key] == got[1][1][key], key


@pytest.mark.parametrize("pieces", [[96], [107], [64, 64], [70, 80], [100, 64, 3]])
def test_ring_trial_enqueue_after_run(pieces, monkeypatch):
    """Spikes listed for the run's last step, straight after the run, are counted and delivered as after the other kernels; at a window's
    first step and inside one, over calls of any length and past the tape's end."""
    b, n, T = 2, 120, sum(pieces)
    wl = synth.ragged_network(n, 40, 60, seed=9, rate_hz=900.0, t=T, b=b, w_mean=0.02, w_std=0.02)
    got = []
    for trials in ("1", "0"):
        monkeypatch.setenv("ADSEQ_RING_TRIALS", trials)
        sim = adseq.Adseq(wl, adseq.RING, 0, batch=b, record_tape=True, max_steps=T - 20)
        cur = torch.zeros((62, b * n), device=sim.dev)
        ids = torch.arange(0, b * n, 3, dtype=torch.int32, device=sim.dev)
        count = torch.tensor([ids.numel()], dtype=torch.int32, device=sim.dev)
        k, seen = 0, []
        for p in pieces:
            sim.run(k, p); k += p
            seen.append(sim.counters())
        # (neurons that did not spike themselves in that step)
        spiked = torch.from_numpy(oracle.Run(wl, adseq.RING, 0, n_steps=T, batch=b).spikes[T - 1].reshape(-1)).to(sim.dev)
        ids = ids[spiked[ids.long()] == 0].contiguous()
        count.fill_(ids.numel())
        sim.enqueue(T - 1, ids, count)
        seen.append(sim.counters())
        for j in range(62):
            sim.deliver(T + j, cur[j])
        seen.append(sim.counters())
        got.append((cur.cpu().numpy(), seen))
        sim.close()
    np.testing.assert_array_equal(got[0][0], got[1][0])
    assert got[1][1][-2]["enqueued"] > got[1][1][-3]["enqueued"] and got[1][1][-1]["delivered"] == got[1][1][-1]["enqueued"]
    for one, many in zip(got[0][1], got[1][1]):
        for key in ("enqueued", "dropped", "delivered", "sum_enqueued", "sum_dropped", "sum_delivered", "tape_spikes"):
            assert one[key] == many[key], key


def _capture(*calls):
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        for fn, args in calls:
            fn(*args)
    return graph


def _same(sim, ref, T):
    torch.cuda.synchronize()
    c, rc = sim.counters(), ref.counters()
    for key in ("enqueued", "dropped", "delivered", "sum_enqueued", "sum_dropped", "sum_delivered"):
        assert c[key] == rc[key], key
    assert c["error_bits"] & ~64 == 0 and c["tape_spikes"] == ref.spikes.sum()
    np.testing.assert_array_equal(sim.membrane_tape(T).cpu().numpy().view(np.uint32), ref.U.view(np.uint32))


@pytest.mark.parametrize("n,b", [(120, 2), (1000, 3)])
@pytest.mark.parametrize("pieces", [[107], [50, 57], [40, 67], [32, 40, 35]])
def test_ring_trial_and_graph_replay(pieces, n, b):
    """Replays of a captured {reset, run} in between eager runs of the same handle, whatever kernels either of them takes: every replay
    and every eager run leaves the oracle's counters and trace, and single steps go on from there."""
    T, more = 107, 30
    wl = synth.ragged_network(n, 40, 30, seed=9, rate_hz=900.0, t=T, b=b, w_mean=0.02, w_std=0.02)
    ref, longer = (oracle.Run(wl, adseq.RING, 0, n_steps=t, batch=b) for t in (T, T + more))
    sim = adseq.Adseq(wl, adseq.RING, 0, batch=b, record_tape=True, max_steps=T + more)
    sim.run(0, T)
    _same(sim, ref, T)
    k, calls = 0, [(sim.reset, ())]
    for p in pieces:
        calls.append((sim.run, (k, p))); k += p
    graph = _capture(*calls)
    for cut in (T, 40, T):
        sim.reset()
        sim.run(0, cut)
        if cut < T:
            sim.run(cut, T - cut)
        _same(sim, ref, T)
        sim.membrane_tape(T).zero_()
        graph.replay()
        _same(sim, ref, T)
        for j in range(more):
            sim.step(T + j)
        _same(sim, longer, T + more)
    sim.close()


@pytest.mark.parametrize("n,b", [(120, 2), (1000, 3), (63, 1)])
@pytest.mark.parametrize("first,second", [([80], 30), ([32, 16, 32], 30), ([80], 90), ([40, 40], 90)])
def test_ring_trial_runs_go_on_after_a_replay(first, second, n, b):
    """A captured run that begins where an eager one ended, and eager runs that begin where a replay ended, by either forward kernel."""
    T = 200
    wl = synth.ragged_network(n, 40, 30, seed=9, rate_hz=900.0, t=T, b=b, w_mean=0.02, w_std=0.02)
    ref = oracle.Run(wl, adseq.RING, 0, n_steps=T, batch=b)
    sim = adseq.Adseq(wl, adseq.RING, 0, batch=b, record_tape=True, max_steps=T)
    sim.run(0, 80)
    graph = _capture((sim.run, (80, second)))
    for _ in range(2):   # (the handle itself does not know of the steps of a replay)
        sim.reset()
        k = 0
        for p in first:
            sim.run(k, p); k += p
        graph.replay()
        torch.cuda.synchronize()
        assert sim.counters()["error_bits"] & ~64 == 0
        np.testing.assert_array_equal(sim.membrane_tape(80 + second).cpu().numpy().view(np.uint32), ref.U[:80 + second].view(np.uint32))
    sim.reset()
    calls, k = [(sim.reset, ())], 0
    for p in first + [second]:
        calls.append((sim.run, (k, p))); k += p
    graph = _capture(*calls)
    for tail in ([T - k], [10] * ((T - k) // 10)):
        for fn, args in calls:
            fn(*args)
        graph.replay()
        at = k
        for p in tail:
            sim.run(at, p); at += p
        _same(sim, ref, T)
    sim.close()
