"""Open-loop stretches of the ring (adseq_run_open: all the steps of a window enqueued in one launch and popped in
another) against the oracle, bit for bit: calls cut so that stretches start and end anywhere in a window, mixed with
single deliver / enqueue calls; output rows that are apart, that share one buffer and that overlap."""
import ctypes as C

import numpy as np
import pytest
import torch

from oracle import oracle
from paper_2512_05906_amd import adseq, synth

pytestmark = pytest.mark.gpu


def _lists(wl, B, T, seed, rate):
    rng = np.random.default_rng(seed)
    forced = (rng.random((T, B * wl.n_neurons)) < rate).astype(np.uint8)
    forced[5] = 0
    lists = [np.flatnonzero(forced[n]).astype(np.int32) for n in range(T)]
    return forced.reshape(T, B, wl.n_neurons), lists


@pytest.mark.parametrize("n,fan,b,d_max,window", [(301, 40, 3, 37, 16), (1, 5, 1, 3, 16), (70000, 6, 1, 20, 16), (500, 30, 2, 70, 64), (130, 20, 1, 9, 4)])
@pytest.mark.parametrize("stride", ["apart", "wide", "one", "overlap"])
def test_open_stretches(n, fan, b, d_max, window, stride, monkeypatch):
    monkeypatch.setenv("ADSEQ_RING_WINDOW", str(window))
    T = 150
    wl = synth.ragged_network(n, fan, d_max, seed=n + b, rate_hz=0.0, t=T, b=b, w_mean=0.01, w_std=0.02)
    bn = b * n
    forced, lists = _lists(wl, b, T, seed=3, rate=0.02 if n < 10000 else 0.002)
    ref = oracle.Run(wl, oracle.RING, 0, n_steps=T, batch=b, forced_spikes=forced, keep_currents=True)
    want = ref.Iq.reshape(T, bn).astype(np.float32) * np.float32(2.0 ** -24)
    sim = adseq.Adseq(wl, adseq.RING, 0, batch=b)
    counts = torch.tensor([len(x) for x in lists], dtype=torch.int32, device=sim.dev)
    offs = np.concatenate([[0], np.cumsum([len(x) for x in lists])]).astype(np.int64)
    ids = torch.from_numpy(np.concatenate(lists + [np.zeros(1, np.int32)])).to(sim.dev)
    step = {"apart": bn, "wide": bn + 5, "one": 0, "overlap": max(1, bn - 1)}[stride]
    s = 0
    for piece in (1, 2, 3, 20, "d", 30, 64, 29):
        if piece == "d":
            out = torch.zeros(bn, dtype=torch.float32, device=sim.dev)
            sim.deliver(s, out); sim.enqueue(s, ids[int(offs[s]):], counts[s:])
            np.testing.assert_array_equal(out.cpu().numpy().view(np.uint32), want[s].view(np.uint32))
            s += 1
            continue
        buf = torch.zeros((piece - 1) * step + bn, dtype=torch.float32, device=sim.dev)
        sim.run_open(s, piece, ids, offs[s:s + piece], counts[s:], buf, step)
        exp = np.zeros((piece - 1) * step + bn, np.float32)
        for k in range(piece):
            exp[k * step:k * step + bn] = want[s + k]
        np.testing.assert_array_equal(buf.cpu().numpy().view(np.uint32), exp.view(np.uint32))
        s += piece
    assert s == T
    c, rc = sim.counters(), ref.counters()
    for key in ("enqueued", "dropped", "delivered", "sum_enqueued", "sum_dropped", "sum_delivered"):
        assert c[key] == rc[key], key
    sim.close()


@pytest.mark.parametrize("kind,cap", [(adseq.FIFO, 1), (adseq.FIFO, 5), (adseq.FIFO, 40), (adseq.SORTED, 1), (adseq.SORTED, 7)])
@pytest.mark.parametrize("n,fan,b,d_max,rate,steps", [(301, 200, 2, 37, 0.05, "16"), (1, 5, 1, 3, 0.5, "16"), (3000, 8, 1, 1, 0.02, "16"), (130, 40, 3, 20, 0.1, "2")])
@pytest.mark.parametrize("stride", ["apart", "one", "overlap"])
def test_open_stretches_bounded(kind, cap, n, fan, b, d_max, rate, steps, stride, monkeypatch):
    """FIFO and SORTED: the steps of a stretch registered in one launch and taken through by the targets' owners in another
    (k_fanout_steps, k_queue_steps); queues that overflow, more contenders in a step than record slots (301 x 200), delays of
    one step only; a second enqueue for the last step of a stretch, whose events are admitted together with the first's."""
    monkeypatch.setenv("ADSEQ_QUEUE_STEPS", steps)
    T = 120
    wl = synth.ragged_network(n, fan, d_max, seed=n + b, rate_hz=0.0, t=T, b=b, w_mean=0.01, w_std=0.02)
    bn = b * n
    forced, lists = _lists(wl, b, T, seed=4, rate=rate)
    ref = oracle.Run(wl, kind, cap, n_steps=T, batch=b, forced_spikes=forced, keep_currents=True)
    want = ref.Iq.reshape(T, bn).astype(np.float32) * np.float32(2.0 ** -24)
    sim = adseq.Adseq(wl, kind, cap, batch=b)
    step = {"apart": bn, "one": 0, "overlap": max(1, bn - 1)}[stride]
    half = [len(x) // 2 for x in lists]
    s = 0
    for piece in (1, 3, 4, 20, 33, 2, 57):
        # (the last step's list in two parts: the second part comes by an enqueue of its own)
        lens = [len(x) for x in lists[s:s + piece]]
        lens[-1] = half[s + piece - 1]
        ids = torch.from_numpy(np.concatenate(lists[s:s + piece] + [np.zeros(1, np.int32)])).to(sim.dev)
        offs = np.concatenate([[0], np.cumsum([len(x) for x in lists[s:s + piece]])]).astype(np.int64)
        counts = torch.tensor(lens + [len(lists[s + piece - 1]) - lens[-1]], dtype=torch.int32, device=sim.dev)
        buf = torch.zeros((piece - 1) * step + bn, dtype=torch.float32, device=sim.dev)
        sim.run_open(s, piece, ids, offs[:piece], counts, buf, step)
        sim.enqueue(s + piece - 1, ids[int(offs[piece - 1]) + lens[-1]:], counts[piece:])
        exp = np.zeros((piece - 1) * step + bn, np.float32)
        for k in range(piece):
            exp[k * step:k * step + bn] = want[s + k]
        np.testing.assert_array_equal(buf.cpu().numpy().view(np.uint32), exp.view(np.uint32))
        s += piece
    assert s == T
    c, rc = sim.counters(), ref.counters()
    for key in ("enqueued", "dropped", "delivered", "sum_enqueued", "sum_dropped", "sum_delivered"):
        assert c[key] == rc[key], key
    sim.close()


def _launches(call):
    """Kernels that a call launches: nodes of the graph that it is captured into."""
    graph = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(graph):
        call()
    lib = [line.split()[-1] for line in open("/proc/self/maps") if "libamdhip64.so" in line][0]
    n = C.c_size_t(0)
    assert C.CDLL(lib).hipGraphGetNodes(C.c_void_p(graph.raw_cuda_graph()), None, C.byref(n)) == 0
    return n.value


@pytest.mark.parametrize("kind,cap", [(adseq.FIFO, 2), (adseq.SORTED, 2)])
@pytest.mark.parametrize("n,rate,crowded", [(5000, 0.2, True), (150, 0.6, True), (5000, 0.02, False)])
def test_crowded_stretches_go_step_by_step(kind, cap, n, rate, crowded):
    """More events in a step than 65,536, or than there are record slots: two launches per step; otherwise two per stretch,
    the spikes' rows spread over as many blocks as a step's.  In between, calls of either sort in turn, against the oracle."""
    T = 90
    wl = synth.ragged_network(n, 150 if crowded else 30, 25, seed=n, rate_hz=0.0, t=T, b=1, w_mean=0.01, w_std=0.02)
    rng = np.random.default_rng(2)
    dense = (np.arange(T) // 30) != 1   # (30 crowded steps, 30 sparse ones, 30 crowded ones)
    forced = (rng.random((T, n)) < np.where(dense, rate, 0.01)[:, None]).astype(np.uint8)
    ref = oracle.Run(wl, kind, cap, n_steps=T, batch=1, forced_spikes=forced.reshape(T, 1, n), keep_currents=True)
    sim = adseq.Adseq(wl, kind, cap)
    counts = torch.from_numpy(forced.sum(axis=1).astype(np.int32)).to(sim.dev)
    offs = np.concatenate([[0], np.cumsum(forced.sum(axis=1))]).astype(np.int64)
    ids = torch.from_numpy(np.flatnonzero(forced).astype(np.int32) % n).to(sim.dev)
    out = torch.zeros((T, n), dtype=torch.float32, device=sim.dev)
    sim.run_open(0, T, ids, offs[:T], counts, out, n)
    want = ref.Iq.reshape(T, n).astype(np.float32) * np.float32(2.0 ** -24)
    np.testing.assert_array_equal(out.cpu().numpy().view(np.uint32), want.view(np.uint32))
    c, rc = sim.counters(), ref.counters()
    for key in ("enqueued", "dropped", "delivered", "sum_enqueued", "sum_dropped", "sum_delivered"):
        assert c[key] == rc[key], key
    sim.reset()
    torch.cuda.synchronize()
    # (29 steps in stretches, the last one in two launches; or all 30 in two each)
    assert _launches(lambda: sim.run_open(0, 30, ids, offs[:30], counts, out, n)) == (60 if crowded else 4)
    sim.close()


@pytest.mark.parametrize("kind,cap", [(adseq.FIFO, 1), (adseq.FIFO, 40), (adseq.SORTED, 3)])
@pytest.mark.parametrize("n,fan,b,d_max,events,steps", [(3001, 1, 1, 80, 0.001, "512"), (700, 30, 3, 37, 0.05, "512"), (1, 5, 1, 3, 0.05, "128"),
                                                        (97, 250, 1, 250, 0.06, "256")])
@pytest.mark.parametrize("stride", ["apart", "odd", "one"])
def test_stretches_of_short_rows(kind, cap, n, fan, b, d_max, events, steps, stride, monkeypatch):
    """k_fanout_lanes and k_queue_events (events: per target and step): stretches of up to 512 steps, events in the first and the last
    step of a 64-step group, several contenders in a step, rows shorter and longer than a wavefront, output rows on any alignment,
    and what an enqueue adds to the last step; two runs of the handle."""
    monkeypatch.setenv("ADSEQ_QUEUE_STEPS", steps)
    T = 1100
    wl = synth.ragged_network(n, fan, d_max, seed=n + b, rate_hz=0.0, t=T, b=b, w_mean=0.01, w_std=0.02)
    bn = b * n
    rng = np.random.default_rng(9)
    forced = (rng.random((T, bn)) < 1.5 * events / max(1.0, wl.n_synapses / n)).astype(np.uint8)
    forced[[0, 63, 64, 127, 128, 511, 512]] |= (rng.random((7, bn)) < min(1.0, 2.0 / bn)).astype(np.uint8)
    forced[200:230] = 0
    lists = [np.flatnonzero(x).astype(np.int32) for x in forced]
    ref = oracle.Run(wl, kind, cap, n_steps=T, batch=b, forced_spikes=forced.reshape(T, b, n), keep_currents=True)
    want = ref.Iq.reshape(T, bn).astype(np.float32) * np.float32(2.0 ** -24)
    sim = adseq.Adseq(wl, kind, cap, batch=b)
    step = {"apart": bn, "odd": bn + 3, "one": 0}[stride]
    ids = torch.from_numpy(np.concatenate(lists + [np.zeros(1, np.int32)])).to(sim.dev)
    offs = np.concatenate([[0], np.cumsum([len(x) for x in lists])]).astype(np.int64)
    for _ in range(2):
        sim.reset()
        s = 0
        for piece in (65, 66, 600, 20, T - 751):
            lens = [len(x) for x in lists[s:s + piece]]
            half = lens[-1] // 2
            counts = torch.tensor(lens[:-1] + [half, lens[-1] - half], dtype=torch.int32, device=sim.dev)
            buf = torch.full(((piece - 1) * step + bn + 1,), 7.0, dtype=torch.float32, device=sim.dev)
            out = buf[1:] if stride == "odd" else buf[:-1]     # (rows that begin anywhere on four bytes)
            sim.run_open(s, piece, ids, offs[s:s + piece], counts, out, step)
            sim.enqueue(s + piece - 1, ids[int(offs[s + piece - 1]) + half:], counts[piece:])
            exp = np.full((piece - 1) * step + bn, 7.0, np.float32)
            for k in range(piece):
                exp[k * step:k * step + bn] = want[s + k]
            np.testing.assert_array_equal(out.cpu().numpy().view(np.uint32), exp.view(np.uint32))
            s += piece
        assert s == T
        c, rc = sim.counters(), ref.counters()
        for key in ("enqueued", "dropped", "delivered", "sum_enqueued", "sum_dropped", "sum_delivered"):
            assert c[key] == rc[key], key
    sim.close()


@pytest.mark.parametrize("kind,cap", [(adseq.FIFO, 3), (adseq.SORTED, 6)])
@pytest.mark.parametrize("n,fan,b,same", [(301, 40, 2, 200), (90, 3, 1, 90), (4000, 2, 1, 17)])
def test_steps_that_share_one_list(kind, cap, n, fan, b, same, monkeypatch):
    """Every step of a call has the same spikes, listed once: the positions of the lists do not say how many there are."""
    T = 140
    wl = synth.ragged_network(n, fan, 30, seed=n, rate_hz=0.0, t=T, b=b, w_mean=0.01, w_std=0.02)
    lists = [np.random.default_rng(k).choice(b * n, same, replace=False).astype(np.int32) for k in range(5)]
    sims = [adseq.Adseq(wl, kind, cap, batch=b) for _ in range(2)]
    out = [torch.zeros((T, b * n), dtype=torch.float32, device=s.dev) for s in sims]
    counts = torch.full((T,), same, dtype=torch.int32, device=sims[0].dev)
    at = 0
    for piece, ids in zip((100, 4, 5, 30, 1), lists):
        ids = torch.from_numpy(ids).to(sims[0].dev)
        sims[0].run_open(at, piece, ids, np.zeros(piece, np.int64), counts, out[0][at], b * n)
        for k in range(piece):
            sims[1].deliver(at + k, out[1][at + k])
            sims[1].enqueue(at + k, ids, counts)
        at += piece
    assert at == T and torch.equal(out[0].view(torch.int32), out[1].view(torch.int32)) and bool((out[0] != 0).any())
    assert sims[0].counters() == sims[1].counters()
    for s in sims:
        s.close()
