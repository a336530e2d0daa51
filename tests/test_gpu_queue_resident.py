"""FIFO and SORTED, closed loop, many steps in one launch (k_queue_run) against the oracle: trace bit for bit, counters,
which events were admitted and dropped, gradients; one, four and eight targets per thread, one block and many, odd sizes,
queues that overflow, more contenders for a target than record slots, rows and bursts of more pieces than are shared out at
once, synaptic states, runs cut into pieces and mixed with single steps, and agreement with two launches per step."""
import numpy as np
import pytest
import torch

from oracle import oracle
from paper_2512_05906_amd import adseq, synth
from tests import helpers as H

pytestmark = pytest.mark.gpu


def _run(wl, kind, cap, T, b, pieces, record=True, **kw):
    sim = adseq.Adseq(wl, kind, cap, batch=b, record_tape=record, max_steps=T, **kw)
    n = 0
    for p in pieces:
        if p == "s":
            sim.step(n); n += 1
        else:
            sim.run(n, p); n += p
    assert n == T
    torch.cuda.synchronize()
    return sim


@pytest.mark.parametrize("kind,cap", [(adseq.FIFO, 1), (adseq.FIFO, 6), (adseq.FIFO, 40), (adseq.SORTED, 1), (adseq.SORTED, 9)])
@pytest.mark.parametrize("n,b,T,d_max,fan,rate,tau_syn,tau_rise,continuous,blocks", [
    (701, 3, 80, 40, 200, 900.0, 0.0, 0.0, False, ""), (100, 1, 60, 1, 60, 900.0, 0.0, 0.0, False, ""),
    (1501, 4, 50, 30, 90, 900.0, 5.0, 0.0, True, "8"), (4100, 4, 40, 20, 40, 900.0, 5.0, 1.0, False, "8"),
    (1100, 8, 24, 12, 2500, 1500.0, 0.0, 0.0, False, "8")])
def test_queue_resident(kind, cap, n, b, T, d_max, fan, rate, tau_syn, tau_rise, continuous, blocks, monkeypatch):
    if blocks:   # (few blocks: four and eight targets per thread)
        monkeypatch.setenv("ADSEQ_QUEUE_BLOCKS", blocks)
    wl = synth.ragged_network(n, fan, d_max, seed=n, rate_hz=rate, t=T, b=b, w_mean=0.6 / fan, w_std=0.6 / fan, continuous=continuous)
    wl.tau_syn_ms, wl.tau_rise_ms = tau_syn, tau_rise
    ref = oracle.Run(wl, kind, cap, n_steps=T, batch=b, n_threads=8)
    assert ref.spikes.sum() > 50
    kw = dict(tape_spike_capacity=T * b * n // 2, tape_event_capacity=T * b * wl.n_synapses // 4)
    rc = ref.counters()
    dc = np.random.default_rng(n).normal(0, 1e-3, (b, n)).astype(np.float32)
    gw, gd = ref.backward(dc, None)
    for resident, pieces, record in (("1", [T], True), ("1", [3, 9, "s", T - 13], True), ("1", [T], False), ("0", [T], True)):
        monkeypatch.setenv("ADSEQ_QUEUE_RESIDENT", resident)
        sim = _run(wl, kind, cap, T, b, pieces, record, **(kw if record else {}))
        c = sim.counters()
        for key in ("enqueued", "dropped", "delivered", "sum_enqueued", "sum_dropped", "sum_delivered"):
            assert c[key] == rc[key], key
        assert c["error_bits"] & ~64 == 0
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


@pytest.mark.parametrize("kind,cap", [(adseq.FIFO, 2), (adseq.SORTED, 3)])
def test_queue_resident_admission_flags_and_reset(kind, cap):
    """Every recorded spike once, every event with its own flag; the same after a reset."""
    T, b = 50, 2
    wl = synth.ragged_network(300, 80, 20, seed=5, rate_hz=900.0, t=T, b=b, w_mean=0.01, w_std=0.01)
    ref = oracle.Run(wl, kind, cap, n_steps=T, batch=b, log_events=True)
    sim = _run(wl, kind, cap, T, b, [T])
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
    sim.close()


@pytest.mark.parametrize("kind,cap", [(adseq.FIFO, 4), (adseq.FIFO, 40), (adseq.SORTED, 4)])
@pytest.mark.parametrize("n,blocks", [(40000, "256"), (16000, "16"), (40000, "16")])
@pytest.mark.parametrize("record", [True, False])
def test_queue_resident_is_what_runs(kind, cap, n, blocks, record, monkeypatch):
    """Every instance -- one, four and eight targets per thread, FIFO slots in LDS and not, with a tape and without -- is
    reached: with one poll per wait its waits run out, and a launch pair per step has none."""
    monkeypatch.setenv("ADSEQ_QUEUE_BLOCKS", blocks)
    monkeypatch.setenv("ADSEQ_RING_RESIDENT_SPINS", "1")
    wl = synth.ragged_network(n, 30, 20, seed=45, rate_hz=700.0, t=40, b=1, w_mean=0.02, w_std=0.01)
    for resident in ("1", "0"):
        monkeypatch.setenv("ADSEQ_QUEUE_RESIDENT", resident)
        sim = _run(wl, kind, cap, 40, 1, [40], record)
        assert (sim.counters()["error_bits"] & 32 != 0) == (resident == "1")
        sim.close()


def test_queue_resident_wait_that_runs_out_is_reported(monkeypatch):
    """Failure path of the bounded waits, forced from the host (one poll per wait): the kernel runs to its end, the error
    word carries bit 32, a reset clears it."""
    monkeypatch.setenv("ADSEQ_RING_RESIDENT_SPINS", "1")
    wl = synth.ragged_network(40000, 30, 20, seed=45, rate_hz=700.0, t=60, b=1, w_mean=0.02, w_std=0.01)
    sim = _run(wl, adseq.FIFO, 4, 60, 1, [60])
    assert sim.counters()["error_bits"] & 32
    with pytest.raises(adseq.AdseqError):
        sim.drop_count()
    sim.reset()
    assert sim.counters()["error_bits"] == 0
    sim.close()


def test_waits_outlast_foreign_kernels(monkeypatch):
    """The bounded kinds' waits last for a second and more, not tens of ms, before a run is void: a foreign kernel may hold compute
    units that long.  (Cells withheld from the host: the reverse sweep's waits run out, its kernels end.)"""
    monkeypatch.setenv("ADSEQ_RING_FLOW_WITHHOLD", "1")
    T = 30
    wl = synth.ragged_network(3000, 30, 20, seed=45, rate_hz=900.0, t=T, b=1, w_mean=0.02, w_std=0.01)
    sim = _run(wl, adseq.FIFO, 4, T, 1, [T])
    g = torch.empty(wl.n_synapses, device=sim.dev)
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    a.record()
    sim.backward(torch.full((3000,), 1e-3, device=sim.dev), None, g, g.clone())
    b.record()
    torch.cuda.synchronize()
    assert sim.counters()["error_bits"] & 32
    assert 300.0 < a.elapsed_time(b) < 30000.0
    sim.close()


@pytest.mark.parametrize("kind,cap,n,b", [(adseq.SORTED, 128, 16000, 1), (adseq.FIFO, 32, 16000, 1), (adseq.FIFO, 128, 40000, 5),
                                          (adseq.SORTED, 12, 40000, 15)])
def test_bursts(kind, cap, n, b, monkeypatch):
    """25 contenders per target in every step, room for all of them, for some and for none: same trace, counters and (through
    the flags) gradients as a launch pair per step, and not slower by more than half where one target per thread is."""
    T = 16
    rng = np.random.default_rng(3)
    fan = 100
    wl = synth.Workload(name="bursts", n_neurons=n, fan_out=fan, n_steps=T, batch=b, d_max_steps=4, ext_rate_hz=2500.0,
                        ext_weight=1.5, seed=3, row_ptr=np.arange(0, n * fan + 1, fan, dtype=np.int64),
                        col=rng.integers(0, n, n * fan).astype(np.int32), weight=rng.normal(0, 1e-3, n * fan).astype(np.float32))
    wl.delay_steps = rng.integers(1, 5, n * fan).astype(np.uint8)
    dc = torch.full((b * n,), 1e-3, device="cuda:0")
    got = []
    for resident in ("1", "0"):
        monkeypatch.setenv("ADSEQ_QUEUE_RESIDENT", resident)
        sim = adseq.Adseq(wl, kind, cap, record_tape=True, max_steps=T, tape_spike_capacity=b * n * T // 3)
        a, e = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        ms = []
        for _ in range(3):
            sim.reset()
            torch.cuda.synchronize()
            a.record()
            sim.run(0, T)
            e.record()
            torch.cuda.synchronize()
            ms.append(a.elapsed_time(e))
        g = [torch.empty(wl.n_synapses, device=sim.dev) for _ in range(2)]
        sim.backward(dc, None, *g)
        got.append((min(ms), sim.counters(), sim.tape()["U"].cpu().numpy().view(np.uint32).copy(), [x.cpu().numpy() for x in g]))
        sim.close()
    (ms1, c1, U1, g1), (ms0, c0, U0, g0) = got
    assert c1 == c0 and c1["error_bits"] & ~64 == 0 and c1["tape_spikes"] > b * n * T // 5
    assert (c1["dropped"] > 0) == (cap < 128)
    np.testing.assert_array_equal(U1, U0)
    for x, y in zip(g1, g0):
        H.grad_close(x, y)
    assert n * b > 16000 or ms1 < 1.5 * ms0


@pytest.mark.parametrize("cap", [2, 7, 8, 9, 16, 17, 40])
@pytest.mark.parametrize("resident", ["1", "0"])
def test_sorted_insertion(cap, resident, monkeypatch):
    """Ordered queues around the eight slots that an insertion moves at a time: front, middle and end, equal arrival steps,
    full queues, the array's end anywhere (its front goes round many times)."""
    monkeypatch.setenv("ADSEQ_QUEUE_RESIDENT", resident)
    T, b = 300, 2
    wl = synth.ragged_network(90, 60, 30, seed=cap, rate_hz=600.0, t=T, b=b, w_mean=0.004, w_std=0.01)
    ref = oracle.Run(wl, adseq.SORTED, cap, n_steps=T, batch=b, n_threads=8)
    sim = _run(wl, adseq.SORTED, cap, T, b, [T], tape_spike_capacity=T * b * 90 // 2)
    c, rc = sim.counters(), ref.counters()
    for key in ("enqueued", "dropped", "delivered", "sum_enqueued", "sum_dropped", "sum_delivered"):
        assert c[key] == rc[key], key
    assert rc["delivered"] > 5 * cap * b * 90 and (rc["dropped"] > 0) == (cap < 40)
    np.testing.assert_array_equal(sim.tape()["U"].cpu().numpy().view(np.uint32), ref.U.view(np.uint32))
    sim.close()
