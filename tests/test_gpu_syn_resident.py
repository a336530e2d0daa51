"""One queue per synapse, closed loop, many steps in one launch (k_syn_run) against the oracle: trace bit for bit, counters, which
events were admitted, replaced and dropped, gradients; one and four neurons per thread, rows whose front does not fit LDS, masks of
one delay word and of several, runs cut into pieces, mixed with single steps and with the queue entry points, and agreement with
three launches per step."""
import numpy as np
import pytest
import torch

from oracle import oracle
from paper_2512_05906_amd import adseq, synth
from tests import helpers as H

pytestmark = pytest.mark.gpu
KINDS = [(adseq.SYN_FIFO, 1), (adseq.SYN_FIFO, 3), (adseq.SYN_LATEST, 1), (adseq.SYN_BINS, 1), (adseq.SYN_BINS, 3), (adseq.SYN_BINS, 8)]


def _run(wl, kind, cap, T, b, pieces, **kw):
    sim = adseq.Adseq(wl, kind, cap, batch=b, record_tape=True, max_steps=T, **kw)
    n = 0
    for p in pieces:
        if p == "s":
            sim.step(n); n += 1
        else:
            sim.run(n, p); n += p
    assert n == T
    torch.cuda.synchronize()
    return sim


@pytest.mark.parametrize("kind,cap", KINDS)
@pytest.mark.parametrize("n,b,T,d_max,fan,rate,gain,tau_syn,tau_rise,continuous,blocks", [
    (701, 3, 80, 40, 200, 900.0, 0.6, 0.0, 0.0, False, ""), (100, 1, 60, 1, 60, 900.0, 0.6, 0.0, 0.0, False, ""),
    (63, 1, 300, 130, 40, 900.0, 1.5, 0.0, 0.0, False, ""), (200, 2, 270, 64, 30, 2500.0, 0.5, 0.0, 0.0, False, ""),
    (1501, 4, 50, 30, 150, 900.0, 0.6, 5.0, 0.0, True, "8"), (4100, 4, 40, 20, 40, 900.0, 0.6, 5.0, 1.0, False, "16"),
    (1100, 8, 24, 8, 2500, 1500.0, 0.6, 0.0, 0.0, False, "8"), (300, 2, 60, 2, 40, 2500.0, 0.6, 0.0, 0.0, False, ""),
    (300, 2, 60, 3, 40, 2500.0, 0.03, 5.0, 1.0, False, ""), (300, 2, 60, 4, 40, 2500.0, 0.6, 0.0, 0.0, False, "")])
def test_syn_resident(kind, cap, n, b, T, d_max, fan, rate, gain, tau_syn, tau_rise, continuous, blocks, monkeypatch):
    if blocks:   # (few blocks: four neurons per thread)
        monkeypatch.setenv("ADSEQ_SYN_BLOCKS", blocks)
    wl = synth.ragged_network(n, fan, d_max, seed=n, rate_hz=rate, t=T, b=b, w_mean=gain / fan, w_std=gain / fan, continuous=continuous)
    wl.tau_syn_ms, wl.tau_rise_ms = tau_syn, tau_rise
    ref = oracle.Run(wl, kind, cap, n_steps=T, batch=b, n_threads=8)
    assert ref.spikes.sum() > 50
    kw = dict(tape_spike_capacity=T * b * n // 2, tape_event_capacity=T * b * wl.n_synapses // 2)
    rc = ref.counters()
    if d_max > 50:
        assert rc["dropped"] > 0 or cap == 8
    dc = np.random.default_rng(n).normal(0, 1e-3, (b, n)).astype(np.float32)
    gw, gd = ref.backward(dc, None)
    for resident, pieces in (("1", [T]), ("1", [3, 9, T - 12]), ("1", [T // 2, "s", T - 1 - T // 2]), ("0", [T])):
        monkeypatch.setenv("ADSEQ_SYN_RESIDENT", resident)
        sim = _run(wl, kind, cap, T, b, pieces, **kw)
        c = sim.counters()
        for key in ("enqueued", "dropped", "delivered", "sum_enqueued", "sum_dropped", "sum_delivered"):
            assert c[key] == rc[key], (key, resident, pieces)
        assert c["error_bits"] & ~64 == 0 and c["tape_spikes"] == ref.spikes.sum()
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


@pytest.mark.parametrize("kind,cap", [(adseq.SYN_FIFO, 2), (adseq.SYN_LATEST, 1), (adseq.SYN_BINS, 2)])
@pytest.mark.parametrize("pieces", [[200], [140, 60], [70, "s", 129]])
def test_syn_resident_admission_flags_and_reset(kind, cap, pieces):
    """Every recorded spike once, every event with its own flag, also those of steps before the call that replaced them; the same
    after a reset."""
    T, b = 200, 2
    wl = synth.ragged_network(90, 30, 70, seed=5, rate_hz=900.0, t=T, b=b, w_mean=0.03, w_std=0.03)
    ref = oracle.Run(wl, kind, cap, n_steps=T, batch=b, log_events=True)
    sim = _run(wl, kind, cap, T, b, pieces, tape_spike_capacity=T * b * 90, tape_event_capacity=T * b * wl.n_synapses)
    for _ in range(2):
        tp = sim.tape()
        out = {k: tp[k].cpu().numpy() for k in ("step_offset", "spike_id", "event_base")}
        np.testing.assert_array_equal(H.spikes_from_tape(out, wl, b), ref.spikes)
        admitted, dropped = H.gpu_dropped_set(sim, out, wl)
        delivered, want_dropped = H.oracle_sets(ref)
        assert dropped == want_dropped and len(dropped) > 0 and delivered <= admitted
        sim.reset()
        sim.run(0, T)
        torch.cuda.synchronize()


@pytest.mark.parametrize("kind,cap", [(adseq.SYN_FIFO, 2), (adseq.SYN_LATEST, 1), (adseq.SYN_BINS, 3)])
def test_syn_resident_then_queue_entry_points(kind, cap, monkeypatch):
    """What is in flight after a run comes out of the queues step by step as after launches per step, and so do the events pushed on
    top of it."""
    T, b, n = 150, 2, 120
    wl = synth.ragged_network(n, 40, 60, seed=9, rate_hz=900.0, t=T, b=b, w_mean=0.02, w_std=0.02)
    got = []
    for resident in ("1", "0"):
        monkeypatch.setenv("ADSEQ_SYN_RESIDENT", resident)
        sim = _run(wl, kind, cap, T, b, [T])
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


def test_syn_resident_past_the_tape_and_wait_that_runs_out(monkeypatch):
    """The steps beyond the tape go by launches per step; a wait that runs out (one poll) ends the launch and is reported."""
    wl = synth.ragged_network(3000, 40, 20, seed=4, rate_hz=400.0, t=60, b=1, w_mean=0.01, w_std=0.01)
    ref = oracle.Run(wl, adseq.SYN_FIFO, 2, n_steps=60, batch=1)
    sim = adseq.Adseq(wl, adseq.SYN_FIFO, 2, record_tape=True, max_steps=40)
    sim.run(0, 60)
    c, rc = sim.counters(), ref.counters()
    assert (c["enqueued"], c["dropped"], c["delivered"]) == (rc["enqueued"], rc["dropped"], rc["delivered"])
    sim.close()
    monkeypatch.setenv("ADSEQ_RING_RESIDENT_SPINS", "1")
    sim = adseq.Adseq(wl, adseq.SYN_FIFO, 2, record_tape=True, max_steps=60)
    sim.run(0, 60)
    torch.cuda.synchronize()
    assert sim.counters()["error_bits"] & 32
    with pytest.raises(adseq.AdseqError):
        sim.drop_count()
    sim.close()


@pytest.mark.parametrize("kind,cap", [(adseq.SYN_FIFO, 2), (adseq.SYN_FIFO, 3), (adseq.SYN_LATEST, 1), (adseq.SYN_BINS, 3)])
@pytest.mark.parametrize("n,blocks", [(3000, ""), (6000, "8")])
def test_syn_resident_is_what_runs(kind, cap, n, blocks, monkeypatch):
    """Every instance -- one and four neurons per thread, a front of one step and of three -- is reached: with one poll per wait its
    waits run out, and three launches per step have none."""
    if blocks:
        monkeypatch.setenv("ADSEQ_SYN_BLOCKS", blocks)
    monkeypatch.setenv("ADSEQ_RING_RESIDENT_SPINS", "1")
    wl = synth.ragged_network(n, 40, 20, seed=4, rate_hz=400.0, t=60, b=1, w_mean=0.01, w_std=0.01)
    for resident in ("1", "0"):
        monkeypatch.setenv("ADSEQ_SYN_RESIDENT", resident)
        sim = _run(wl, kind, cap, 60, 1, [60])
        assert (sim.counters()["error_bits"] & 32 != 0) == (resident == "1")
        sim.close()


@pytest.mark.parametrize("kind,cap", [(adseq.SYN_FIFO, 1), (adseq.SYN_FIFO, 4), (adseq.SYN_LATEST, 1), (adseq.SYN_BINS, 3)])
@pytest.mark.parametrize("pieces", [[90], [60, 30]])
def test_syn_resident_enqueue_after_run(kind, cap, pieces, monkeypatch):
    """Spikes listed for the run's last step, straight after the run, are admitted, counted and delivered as after launches per step."""
    T, b, n = sum(pieces), 2, 120
    wl = synth.ragged_network(n, 40, 60, seed=9, rate_hz=900.0, t=T, b=b, w_mean=0.02, w_std=0.02)
    # (neurons that did not spike themselves in that step)
    spiked = oracle.Run(wl, kind, cap, n_steps=T, batch=b).spikes[T - 1].reshape(-1)
    listed = np.array([g for g in range(0, b * n, 3) if not spiked[g]], np.int32)
    got = []
    for resident in ("1", "0"):
        monkeypatch.setenv("ADSEQ_SYN_RESIDENT", resident)
        sim = _run(wl, kind, cap, T, b, pieces)
        before = sim.counters()
        sim.enqueue(T - 1, torch.from_numpy(listed).to(sim.dev), torch.tensor([len(listed)], dtype=torch.int32, device=sim.dev))
        seen = [before, sim.counters()]
        cur = torch.zeros((62, b * n), device=sim.dev)
        for j in range(62):
            sim.deliver(T + j, cur[j])
        seen.append(sim.counters())
        got.append((cur.cpu().numpy(), seen))
        sim.close()
    np.testing.assert_array_equal(got[0][0], got[1][0])
    assert got[1][1][1]["enqueued"] > got[1][1][0]["enqueued"]
    assert got[1][1][2]["delivered"] == got[1][1][2]["enqueued"] - got[1][1][2]["dropped"]
    for one, many in zip(got[0][1], got[1][1]):
        for key in ("enqueued", "dropped", "delivered", "sum_enqueued", "sum_dropped", "sum_delivered"):
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


@pytest.mark.parametrize("kind,cap", [(adseq.SYN_FIFO, 2), (adseq.SYN_LATEST, 1), (adseq.SYN_BINS, 3)])
@pytest.mark.parametrize("pieces", [[90], [50, 40]])
def test_syn_resident_and_graph_replay(kind, cap, pieces):
    """Replays of a captured {reset, run} in between eager runs of the same handle: every replay and every eager run leaves the oracle's
    counters and trace, and single steps and runs go on from there; a capture alone changes nothing."""
    T, b, more = 90, 2, 30
    wl = synth.ragged_network(120, 40, 40, seed=9, rate_hz=900.0, t=T, b=b, w_mean=0.02, w_std=0.02)
    ref, longer = (oracle.Run(wl, kind, cap, n_steps=t, batch=b) for t in (T, T + more))
    room = (T + more) * b * wl.n_neurons // 2
    sim = adseq.Adseq(wl, kind, cap, batch=b, record_tape=True, max_steps=T + more, tape_spike_capacity=room,
                      tape_event_capacity=(T + more) * b * wl.n_synapses // 2)
    sim.run(0, T)
    _same(sim, ref, T)
    k, calls = 0, [(sim.reset, ())]
    for p in pieces:
        calls.append((sim.run, (k, p))); k += p
    for captures in range(2):
        graph = _capture(*calls)
        _same(sim, ref, T)
        for single in (True, False):
            graph.replay()
            _same(sim, ref, T)
            for j in range(more if single else 0):
                sim.step(T + j)
            if not single:
                sim.run(T, more)
            _same(sim, longer, T + more)
            sim.reset()
            sim.run(0, T)
            _same(sim, ref, T)
            graph.replay()
            _same(sim, ref, T)
            sim.reset()
            sim.run(0, T)
    sim.close()


@pytest.mark.parametrize("kind,cap", [(adseq.SYN_FIFO, 2), (adseq.SYN_LATEST, 1), (adseq.SYN_BINS, 3)])
def test_syn_resident_then_captured_run(kind, cap):
    """A captured run that begins where an eager one ended, replayed after a run and after single steps."""
    T, b = 60, 2
    wl = synth.ragged_network(120, 40, 40, seed=9, rate_hz=900.0, t=2 * T, b=b, w_mean=0.02, w_std=0.02)
    ref = oracle.Run(wl, kind, cap, n_steps=2 * T, batch=b)
    sim = adseq.Adseq(wl, kind, cap, batch=b, record_tape=True, max_steps=2 * T, tape_spike_capacity=T * b * wl.n_neurons,
                      tape_event_capacity=T * b * wl.n_synapses)
    sim.run(0, T)
    graph = _capture((sim.run, (T, T)))
    graph.replay()
    _same(sim, ref, 2 * T)
    for single in (False, True):
        sim.reset()
        if single:
            for k in range(T):
                sim.step(k)
        else:
            sim.run(0, T)
        graph.replay()
        torch.cuda.synchronize()
        np.testing.assert_array_equal(sim.membrane_tape(2 * T).cpu().numpy().view(np.uint32), ref.U.view(np.uint32))
        # the counters of a handle that knows of the replayed steps
        sim.reset()
        sim.run(0, 2 * T)
        sim.reset()
        sim.run(0, T)
        sim.run(T, T)
        _same(sim, ref, 2 * T)
    sim.close()


@pytest.mark.parametrize("kind,cap", [(adseq.SYN_FIFO, 2), (adseq.SYN_LATEST, 1), (adseq.SYN_BINS, 1), (adseq.SYN_BINS, 3)])
@pytest.mark.parametrize("spikes,events", [(300, 1 << 18), (301, 1 << 18), (1 << 14, 9000), (300, 9000), (1 << 14, 9001)])
def test_syn_resident_full_tape(kind, cap, spikes, events, monkeypatch):
    """A tape whose spike list or admission flags are full in the middle of a run: the counters are exact all the same, and the flags
    those of launches per step."""
    T, b, n = 150, 2, 120
    wl = synth.ragged_network(n, 40, 60, seed=9, rate_hz=900.0, t=T, b=b, w_mean=0.02, w_std=0.02)
    ref = oracle.Run(wl, kind, cap, n_steps=T, batch=b)
    rc = ref.counters()
    assert ref.spikes.sum() > 600 and rc["enqueued"] > 18000 and rc["dropped"] > 1000
    got = []
    for resident in ("0", "1"):
        monkeypatch.setenv("ADSEQ_SYN_RESIDENT", resident)
        sim = adseq.Adseq(wl, kind, cap, batch=b, record_tape=True, max_steps=T, tape_spike_capacity=spikes, tape_event_capacity=events)
        flags = sim.admitted_flags(0, events)
        flags.zero_()
        sim.run(0, T)
        torch.cuda.synchronize()
        c = sim.counters()
        assert c["error_bits"] & ~64 == (4 if spikes < 1000 else 0) + (8 if events < 18000 else 0)
        for key in ("enqueued", "dropped", "delivered", "sum_enqueued", "sum_dropped", "sum_delivered"):
            assert c[key] == rc[key], (key, resident)
        got.append(flags.cpu().numpy())
        sim.close()
    if kind != adseq.SYN_BINS or events > 18000:   # (by launches, a spike without flags of its own leaves those of what it replaces in a bin)
        used = min(events, rc["enqueued"])
        np.testing.assert_array_equal(got[1][:used], got[0][:used])


@pytest.mark.parametrize("kind,cap", [(adseq.SYN_FIFO, 2), (adseq.SYN_LATEST, 1), (adseq.SYN_BINS, 1), (adseq.SYN_BINS, 3)])
@pytest.mark.parametrize("spikes,events", [(300, 1 << 18), (301, 1 << 18), (1 << 14, 9000), (300, 9000), (1 << 14, 9001)])
def test_syn_resident_full_tape_then_steps(kind, cap, spikes, events, monkeypatch):
    """A tape whose spike list or admission flags are full in the middle of a run: single steps on top of it change the flags that they
    would after launches per step, and no byte in front of them."""
    T, b, n, more = 150, 2, 120, 20
    wl = synth.ragged_network(n, 40, 60, seed=9, rate_hz=900.0, t=T, b=b, w_mean=0.02, w_std=0.02)
    ref = oracle.Run(wl, kind, cap, n_steps=T + more, batch=b)
    assert ref.spikes[:T].sum() > 600 and ref.counters()["enqueued"] > 18000
    got = []
    for resident in ("0", "1"):
        monkeypatch.setenv("ADSEQ_SYN_RESIDENT", resident)
        sim = adseq.Adseq(wl, kind, cap, batch=b, record_tape=True, max_steps=T + more, tape_spike_capacity=spikes, tape_event_capacity=events)
        flags = sim.admitted_flags(-64, events + 64)
        flags.zero_()   # (and 64 bytes that nothing lies in)
        sim.run(0, T)
        for k in range(T, T + more):
            sim.step(k)
        torch.cuda.synchronize()
        c, rc = sim.counters(), ref.counters()
        assert c["error_bits"] & 12
        for key in ("enqueued", "dropped", "delivered", "sum_enqueued", "sum_dropped", "sum_delivered"):
            assert c[key] == rc[key], (key, resident)
        got.append(flags.cpu().numpy())
        sim.close()
    np.testing.assert_array_equal(got[1][:64], got[0][:64])
    used = 64 + min(events, int(ref.counters()["enqueued"]))
    if kind != adseq.SYN_BINS or events > 18000:   # (see the test before)
        np.testing.assert_array_equal(got[1][64:used], got[0][64:used])


@pytest.mark.parametrize("cap", [1, 2, 4, 8])
@pytest.mark.parametrize("n,b,T,d_max,fan,rate,blocks", [
    (130, 1, 420, 300, 30, 9900.0, ""),      # 300 held spikes per source: more than a list has room for
    (200, 2, 300, 250, 40, 6000.0, ""), (70, 1, 560, 512, 300, 2500.0, ""), (2500, 1, 150, 140, 20, 6000.0, "8")])
def test_syn_resident_many_spikes(n, b, T, d_max, fan, rate, blocks, cap, monkeypatch):
    """FIFO queues that refuse most of what comes: masks made of many held spikes, more pieces than one look at the rows takes."""
    if blocks:
        monkeypatch.setenv("ADSEQ_SYN_BLOCKS", blocks)
    wl = synth.ragged_network(n, fan, d_max, seed=n, rate_hz=rate, t=T, b=b, w_mean=0.1 / fan, w_std=0.1 / fan, continuous=d_max > 255)
    wl.ext_weight = 1.1
    ref = oracle.Run(wl, adseq.SYN_FIFO, cap, n_steps=T, batch=b, n_threads=8)
    rc = ref.counters()
    assert rc["dropped"] > rc["enqueued"] // 2
    sim = _run(wl, adseq.SYN_FIFO, cap, T, b, [T // 3, T - T // 3], tape_spike_capacity=T * b * n, tape_event_capacity=T * b * wl.n_synapses)
    c = sim.counters()
    for key in ("enqueued", "dropped", "delivered", "sum_enqueued", "sum_dropped", "sum_delivered"):
        assert c[key] == rc[key], key
    assert c["error_bits"] & ~64 == 0
    np.testing.assert_array_equal(sim.tape()["U"].cpu().numpy().view(np.uint32), ref.U.view(np.uint32))
    sim.close()
