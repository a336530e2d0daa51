"""Crowded windows of the ring pulled by the targets (ring_pull.h) against the oracle: trace bit for bit, spike counts, counters and both
gradients.  Parts with a remainder, delays that are no multiple of the window, trials that share spike words, synaptic current
states, more synapses of a part than LDS has room for, runs cut inside windows, and what changes between pulled and staged windows."""
import numpy as np
import pytest
import torch

from oracle import oracle
from paper_2512_05906_amd import adseq, synth

pytestmark = pytest.mark.gpu


def _check(sim, ref):
    torch.cuda.synchronize()
    np.testing.assert_array_equal(sim.tape()["U"].cpu().numpy().view(np.uint32), ref.U.view(np.uint32))
    c, rc = sim.counters(), ref.counters()
    for key in ("enqueued", "dropped", "delivered", "sum_enqueued", "sum_dropped", "sum_delivered"):
        assert c[key] == rc[key], key


@pytest.mark.parametrize("n,b,fan,d_max,T,window,syn", [(2000, 1, 200, 40, 90, 16, 0), (2049, 1, 150, 65, 130, 32, 1), (2500, 1, 300, 33, 80, 16, 2),
                                                        (1501, 2, 90, 33, 90, 16, 0), (901, 3, 120, 70, 150, 32, 1), (6001, 1, 60, 50, 100, 32, 0),
                                                        (2000, 1, 100, 9, 60, 8, 0), (2100, 1, 1600, 40, 70, 32, 0)])
def test_pulled_windows(n, b, fan, d_max, T, window, syn, monkeypatch):
    monkeypatch.setenv("ADSEQ_RING_DENSE", "2")            # every window from the second on
    monkeypatch.setenv("ADSEQ_RING_FORWARD_CHIP", "1")
    monkeypatch.setenv("ADSEQ_RING_WINDOW", str(window))
    monkeypatch.setenv("ADSEQ_RING_BINBLOCKS", "32")
    wl = synth.ragged_network(n, fan, d_max, seed=n, rate_hz=700.0, t=T, b=b, w_mean=1.2 / fan, w_std=1.0 / fan)
    wl.tau_syn_ms, wl.tau_rise_ms = (0.0, 5.0, 5.0)[syn], (0.0, 0.0, 1.0)[syn]
    ref = oracle.Run(wl, oracle.RING, 0, n_steps=T, batch=b, n_threads=8)
    sim = adseq.Adseq(wl, adseq.RING, 0, batch=b, record_tape=True, max_steps=T, step_event_capacity=4000000)
    cut = 2 * window + 3
    for pieces in ([T], [cut, T - cut], [window, 1, 1, T - window - 2]):   # whole, cut inside a window, single steps in between
        sim.reset()
        n0 = 0
        for p in pieces:
            sim.step(n0) if p == 1 else sim.run(n0, p)
            n0 += p
        _check(sim, ref)
        base = -sim.workspace.data_ptr() % 256             # Counters::dense, at byte 76 of the workspace
        assert any(sim.workspace[base + 76:base + 84].cpu().numpy().view(np.uint32).tolist())
    dc = np.random.default_rng(n).normal(0, 1e-3, (b, n)).astype(np.float32)
    gw, gd = ref.backward(dc, None)
    g_w, g_d = torch.empty(wl.n_synapses, device=sim.dev), torch.empty(wl.n_synapses, device=sim.dev)
    sim.backward(torch.from_numpy(dc).to(sim.dev), None, g_w, g_d)
    np.testing.assert_allclose(g_w.cpu().numpy(), gw, rtol=1e-5, atol=1e-6)
    np.testing.assert_allclose(g_d.cpu().numpy(), gd, rtol=1e-5, atol=1e-6)
    sim.close()


def test_from_quiet_to_crowded(monkeypatch):
    """More than 2^21 synapses at the default line: a network that starts quiet and runs away, by staged and then by pulled windows,
    against the same run by staged windows alone (which the other tests hold against the oracle, too slow at this size)."""
    n, fan, d_max, T = 2200, 1000, 60, 400
    wl = synth.ragged_network(n, 4, d_max, seed=5, rate_hz=60.0, t=T, b=1, w_mean=0.0, w_std=0.0)
    rng = np.random.default_rng(5)
    wl.row_ptr = np.arange(n + 1, dtype=np.int64) * fan
    wl.col = rng.integers(0, n, n * fan, dtype=np.int32)
    wl.weight = rng.normal(4.0 / fan, 1.0 / fan, n * fan).astype(np.float32)
    wl.delay_steps = rng.integers(1, d_max + 1, n * fan).astype(np.uint8)
    monkeypatch.setenv("ADSEQ_RING_DENSE", "0")
    ref = adseq.Adseq(wl, adseq.RING, 0, batch=1, record_tape=True, max_steps=T)
    monkeypatch.delenv("ADSEQ_RING_DENSE")
    ref.run(0, T)
    U = ref.tape()["U"]
    per_step = (U.view(T, n) >= wl.v_thresh).sum(dim=1)
    assert per_step[:64].float().mean() < 20 and per_step[-40:].float().mean() > 200
    sim = adseq.Adseq(wl, adseq.RING, 0, batch=1, record_tape=True, max_steps=T)
    base = -sim.workspace.data_ptr() % 256
    crowded = lambda: sim.workspace[base + 76:base + 84].cpu().numpy().view(np.uint32).tolist()
    for cut in (64, 203):   # (the second one inside a window)
        sim.reset()
        sim.run(0, 64)
        assert not any(crowded())
        if cut > 64:
            sim.run(64, cut - 64)
        sim.run(cut, T - cut)
        assert any(crowded())
        assert torch.equal(sim.tape()["U"].view(torch.int32), U.view(torch.int32))
        assert sim.counters() == ref.counters()
    sim.close(); ref.close()


@pytest.mark.parametrize("n,b,fan,d_max,window", [(2000, 1, 200, 40, 16), (1501, 2, 90, 70, 32)])
@pytest.mark.parametrize("stop", ["window", "inside"])
@pytest.mark.parametrize("go_on", ["run", "deliver"])
def test_spikes_listed_after_a_run(n, b, fan, d_max, window, stop, go_on, monkeypatch):
    """Spikes listed on top of the run's last step, the last one of a window or one inside it, travel with the run's own: counted, and
    delivered by the windows that follow, pulled or staged."""
    T = 4 * window + (0 if stop == "window" else 5)
    monkeypatch.setenv("ADSEQ_RING_FORWARD_CHIP", "1")
    monkeypatch.setenv("ADSEQ_RING_WINDOW", str(window))
    monkeypatch.setenv("ADSEQ_RING_BINBLOCKS", "32")
    wl = synth.ragged_network(n, fan, d_max, seed=n, rate_hz=700.0, t=T, b=b, w_mean=1.2 / fan, w_std=1.0 / fan)
    spiked = oracle.Run(wl, oracle.RING, 0, n_steps=T, batch=b, n_threads=8).spikes[T - 1].reshape(-1)
    listed = np.flatnonzero(spiked == 0)[::3].astype(np.int32)     # (neurons that did not spike themselves)
    got = []
    for dense in ("0", "2"):
        monkeypatch.setenv("ADSEQ_RING_DENSE", dense)
        sim = adseq.Adseq(wl, adseq.RING, 0, batch=b, step_event_capacity=4000000)
        ids = torch.from_numpy(listed).to(sim.dev)
        sim.run(0, T)
        seen = [sim.counters()]
        sim.enqueue(T - 1, ids, torch.tensor([len(listed)], dtype=torch.int32, device=sim.dev))
        seen.append(sim.counters())
        at, more = T, 0
        spikes = torch.zeros((4, b * n), dtype=torch.uint8, device=sim.dev)
        if go_on == "run":
            for k in range(4):      # (two windows and a step, whose spikes are handed back)
                sim.run(at, 2 * window)
                sim.step(at + 2 * window, None, spikes[k])
                at += 2 * window + 1
            seen.append(sim.counters())
        cur = torch.zeros((d_max + 1, b * n), device=sim.dev)
        for j in range(d_max + 1):
            sim.deliver(at + j, cur[j])
        seen.append(sim.counters())
        got.append((spikes.cpu().numpy(), cur.cpu().numpy().view(np.uint32), seen))
        sim.close()
    assert got[1][2][1]["enqueued"] > got[1][2][0]["enqueued"] and got[1][2][-1]["delivered"] == got[1][2][-1]["enqueued"]
    np.testing.assert_array_equal(got[0][0], got[1][0])
    np.testing.assert_array_equal(got[0][1], got[1][1])
    assert got[0][2] == got[1][2]


def _kernels(call):
    from torch.profiler import ProfilerActivity, profile
    with profile(activities=[ProfilerActivity.CUDA]) as p:
        call()
        torch.cuda.synchronize()
    return [e.name for e in p.events()]


def _pulled(names):
    return sum("k_win_bin<true, false>" in x for x in names)


@pytest.mark.parametrize("crowded", [0, 1])
def test_one_trial_of_two_is_crowded(crowded, monkeypatch):
    """Two trials, no drive, one of them set off from outside and running away: whichever it is, the windows are pulled from then on, one after the
    other.  Results as by staged windows."""
    n, fan, d_max, T = 2200, 1000, 60, 320
    wl = synth.ragged_network(n, 4, d_max, seed=6, rate_hz=0.0, t=T, b=2, w_mean=0.0, w_std=0.0)
    rng = np.random.default_rng(6)
    wl.row_ptr = np.arange(n + 1, dtype=np.int64) * fan
    wl.col = rng.integers(0, n, n * fan, dtype=np.int32)
    wl.weight = rng.normal(4.0 / fan, 1.0 / fan, n * fan).astype(np.float32)
    wl.delay_steps = rng.integers(1, d_max + 1, n * fan).astype(np.uint8)
    got = []
    for dense in ("0", "1"):
        monkeypatch.setenv("ADSEQ_RING_DENSE", dense)
        sim = adseq.Adseq(wl, adseq.RING, 0, batch=2, record_tape=True, max_steps=T)
        current = torch.zeros((2, n), device=sim.dev)
        current[crowded] = 2.0
        sim.step(0, current)
        sim.run(1, T - 1 - 32)
        base = -sim.workspace.data_ptr() % 256             # Counters::dense, at byte 76 of the workspace
        flags = sim.workspace[base + 76:base + 84].cpu().numpy().view(np.uint32).tolist()
        names = _kernels(lambda: sim.run(T - 32, 32))
        got.append((sim.tape()["U"].clone(), sim.counters()))
        assert dense == "0" or (all(flags) and _pulled(names) == 1), (flags, names)
        sim.close()
    spikes = (got[0][0] >= wl.v_thresh).sum(dim=(0, 2))
    assert int(spikes[crowded]) > 50 * T and int(spikes[1 - crowded]) == 0
    assert torch.equal(got[0][0].view(torch.int32), got[1][0].view(torch.int32)) and got[0][1] == got[1][1]


@pytest.mark.parametrize("n,b,fan,d_max,window", [(2000, 1, 200, 40, 16), (1501, 2, 90, 64, 32)])
def test_which_windows_are_pulled(n, b, fan, d_max, window, monkeypatch):
    """The kernels of a run: every window's expansion may pull where the window words of all the steps its events come from are there, from the
    first window of a run on; after a run that ended inside a window, from the one on that looks no further back than the next boundary."""
    monkeypatch.setenv("ADSEQ_RING_DENSE", "2")
    monkeypatch.setenv("ADSEQ_RING_FORWARD_CHIP", "1")
    monkeypatch.setenv("ADSEQ_RING_WINDOW", str(window))
    windows, back, cut = 12, -(-d_max // window), 2 * window + 3
    T = windows * window
    wl = synth.ragged_network(n, fan, d_max, seed=n, rate_hz=700.0, t=T, b=b, w_mean=1.2 / fan, w_std=1.0 / fan)
    sim = adseq.Adseq(wl, adseq.RING, 0, batch=b, step_event_capacity=4000000)
    names = _kernels(lambda: sim.run(0, T))
    assert _pulled(names) == windows - 1 and not any("k_win_bin<false, false>" in x for x in names)
    sim.reset()
    names = _kernels(lambda: (sim.run(0, cut), sim.run(cut, T - cut)))
    staged = [x for x in names if "k_win_bin<" in x]
    # boundaries 1 and 2 pulled, 3 staged; the words begin again with window 3
    assert ["k_win_bin<true, false>" in x for x in staged] == [k < 3 or k >= 3 + back for k in range(1, windows)]
    sim.close()
