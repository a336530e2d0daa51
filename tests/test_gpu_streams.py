"""Two handles on two streams: runs and reverse sweeps whose kernels each need the whole chip, issued side by side from two
threads without waiting; every result is the oracle's."""
import threading

import numpy as np
import pytest
import torch

from oracle import oracle
from paper_2512_05906_amd import adseq, synth
from tests import helpers as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kinds", [((adseq.FIFO, 4), (adseq.SORTED, 3)), ((adseq.FIFO, 4), (adseq.RING, 0))])
def test_two_streams(kinds):
    T, n = 60, 60000
    wl = synth.ragged_network(n, 12, 20, seed=9, rate_hz=900.0, t=T, b=1, w_mean=0.04, w_std=0.04)
    dc = np.random.default_rng(1).normal(0, 1e-3, (1, n)).astype(np.float32)
    refs = [oracle.Run(wl, k, c, n_steps=T, n_threads=8) for k, c in kinds]
    want = [r.backward(dc, None) for r in refs]
    sims = [adseq.Adseq(wl, k, c, record_tape=True, max_steps=T) for k, c in kinds]
    dcg = torch.from_numpy(dc).to(sims[0].dev)
    grads = [[torch.empty(wl.n_synapses, device=s.dev) for _ in range(2)] for s in sims]
    torch.cuda.synchronize()
    failed = []

    def work(j):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                for _ in range(3):
                    sims[j].reset()
                    sims[j].run(0, T)
                    sims[j].backward(dcg, None, *grads[j])
        except Exception as e:   # (an assertion in a thread would be lost)
            failed.append(e)

    threads = [threading.Thread(target=work, args=(j,)) for j in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    assert not failed
    for j in range(2):
        assert sims[j].counters()["error_bits"] & 32 == 0
        np.testing.assert_array_equal(sims[j].tape()["U"].cpu().numpy().view(np.uint32), refs[j].U.view(np.uint32))
        H.grad_close(grads[j][0].cpu().numpy(), want[j][0])
        H.grad_close(grads[j][1].cpu().numpy(), want[j][1])
        sims[j].close()


@pytest.mark.parametrize("n_ring", [1996, 40000])
def test_ring_waits_for_fifo(n_ring):
    """A FIFO run of 16,000 targets (63 blocks that nearly fill two XCDs), and while it runs a ring of n_ring cells on
    another stream: the ring's run ends after the FIFO's, and both results are the oracle's.  (1,996 cells: the ring's
    kernel on the blocks of one XCD; 40,000: the one over the whole chip.)"""
    T, n = 1500, 16000
    wl = synth.ragged_network(n, 12, 20, seed=9, rate_hz=400.0, t=T, b=1, w_mean=0.04, w_std=0.04)
    small = synth.ragged_network(n_ring, 60, 20, seed=4, rate_hz=400.0, t=T, b=1, w_mean=0.01, w_std=0.01)
    refs = [oracle.Run(wl, adseq.FIFO, 4, n_steps=T, n_threads=8), oracle.Run(small, oracle.RING, 0, n_steps=T, n_threads=8)]
    sims = [adseq.Adseq(wl, adseq.FIFO, 4, record_tape=True, max_steps=T),
            adseq.Adseq(small, adseq.RING, 0, record_tape=True, max_steps=T)]
    streams = [torch.cuda.Stream() for _ in sims]
    ends = [torch.cuda.Event(enable_timing=True) for _ in sims]
    torch.cuda.synchronize()
    for sim, st, end, steps in zip(sims, streams, ends, (T, 40)):
        with torch.cuda.stream(st):
            sim.run(0, steps)
            end.record(st)
    torch.cuda.synchronize()
    assert ends[0].elapsed_time(ends[1]) > 0.0
    with torch.cuda.stream(streams[1]):
        sims[1].run(40, T - 40)
    torch.cuda.synchronize()
    for sim, ref in zip(sims, refs):
        assert sim.counters()["error_bits"] & 32 == 0
        np.testing.assert_array_equal(sim.tape()["U"].cpu().numpy().view(np.uint32), ref.U.view(np.uint32))
        sim.close()


def test_one_handle_value_two_streams():
    """hipStreamPerThread is one handle value and a stream of its own in every thread: a run on the second thread's still
    waits for the one on the first's."""
    per_thread = torch.cuda.ExternalStream(2)
    T = 1500
    wl = synth.ragged_network(16000, 12, 20, seed=9, rate_hz=400.0, t=T, b=1, w_mean=0.04, w_std=0.04)
    sims = [adseq.Adseq(wl, adseq.FIFO, 4, record_tape=True, max_steps=T) for _ in range(2)]
    ends = [torch.cuda.Event(enable_timing=True) for _ in sims]
    torch.cuda.synchronize()
    failed, issued, done = [], threading.Event(), threading.Event()

    def work(j, steps):
        try:
            with torch.cuda.stream(per_thread):
                sims[j].run(0, steps)
                ends[j].record(per_thread)
        except Exception as e:
            failed.append(e)
        issued.set()
        done.wait(60)   # (its stream goes with the thread)

    threads = []
    for j, steps in ((0, T), (1, 40)):
        issued.clear()
        threads.append(threading.Thread(target=work, args=(j, steps)))
        threads[j].start()
        issued.wait(60)
    torch.cuda.synchronize()
    assert not failed
    assert ends[0].elapsed_time(ends[1]) > 0.0
    done.set()
    for t in threads:
        t.join()
    U = [s.tape()["U"].cpu().numpy().view(np.uint32) for s in sims]
    np.testing.assert_array_equal(U[1], U[0][:40])
    for s in sims:
        assert s.counters()["error_bits"] & 32 == 0
        s.close()


@pytest.mark.parametrize("kind,cap", [(adseq.FIFO, 4), (adseq.SORTED, 3), (adseq.SYN_FIFO, 2)])
def test_static_handle_waits_for_nobody(kind, cap, monkeypatch):
    """The static handle takes no turn, so the bounded kinds' runs and reverse sweeps make no launch whose blocks wait for
    one another: with a bound of one poll such a wait would run out (as it does with an ordinary handle)."""
    monkeypatch.setenv("ADSEQ_RING_RESIDENT_SPINS", "1")
    T, n = 60, 3000
    wl = synth.ragged_network(n, 12, 20, seed=9, rate_hz=900.0, t=T, b=1, w_mean=0.04, w_std=0.04)
    dc = np.random.default_rng(1).normal(0, 1e-3, (1, n)).astype(np.float32)
    ref = oracle.Run(wl, kind, cap, n_steps=T, n_threads=8)
    want = ref.backward(dc, None)
    sim = adseq.Adseq(wl, kind, cap, record_tape=True, max_steps=T, static_workspace=True)
    sim.run(0, T)
    grads = [torch.empty(wl.n_synapses, device=sim.dev) for _ in range(2)]
    sim.backward(torch.from_numpy(dc).to(sim.dev), None, *grads)
    torch.cuda.synchronize()
    assert sim.counters()["error_bits"] == 0
    np.testing.assert_array_equal(sim.tape()["U"].cpu().numpy().view(np.uint32), ref.U.view(np.uint32))
    H.grad_close(grads[0].cpu().numpy(), want[0])
    H.grad_close(grads[1].cpu().numpy(), want[1])
    sim.close()


@pytest.mark.parametrize("kind,cap", [(adseq.FIFO, 4), (adseq.SORTED, 3)])
def test_captured_run_waits_for_nobody(kind, cap, monkeypatch):
    """A captured run takes no turn either.  Every replay, with eager work of another handle in between, is the oracle's."""
    monkeypatch.setenv("ADSEQ_RING_RESIDENT_SPINS", "1")
    T, n = 60, 3000
    wl = synth.ragged_network(n, 12, 20, seed=9, rate_hz=900.0, t=T, b=1, w_mean=0.04, w_std=0.04)
    ref = oracle.Run(wl, kind, cap, n_steps=T, n_threads=8)
    sim = adseq.Adseq(wl, kind, cap, record_tape=True, max_steps=T)
    monkeypatch.delenv("ADSEQ_RING_RESIDENT_SPINS")
    other = adseq.Adseq(wl, kind, cap, record_tape=True, max_steps=T)
    U = sim.membrane_tape(T)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        sim.reset()
        sim.run(0, T)
    for _ in range(3):
        U.zero_()
        other.reset()
        other.run(0, T)
        graph.replay()
        torch.cuda.synchronize()
        assert sim.counters()["error_bits"] == 0
        for u in (U, other.membrane_tape(T)):
            np.testing.assert_array_equal(u.cpu().numpy().view(np.uint32).reshape(ref.U.shape), ref.U.view(np.uint32))
    other.close()
    sim.close()


def test_static_ring_takes_its_turn():
    """The static handle's ring waits for the FIFO run of an ordinary handle on another stream, and the other way round."""
    T = 1500
    wl = synth.ragged_network(16000, 12, 20, seed=9, rate_hz=400.0, t=T, b=1, w_mean=0.04, w_std=0.04)
    small = synth.ragged_network(1996, 60, 20, seed=4, rate_hz=400.0, t=T, b=1, w_mean=0.01, w_std=0.01)
    fifo = adseq.Adseq(wl, adseq.FIFO, 4, record_tape=True, max_steps=T)
    ring = adseq.Adseq(small, adseq.RING, 0, record_tape=True, max_steps=1000, static_workspace=True)
    for order in (((fifo, T), (ring, 40)), ((ring, 1000), (fifo, 40))):
        ends = [torch.cuda.Event(enable_timing=True) for _ in order]
        fifo.reset(); ring.reset()
        torch.cuda.synchronize()
        for (sim, steps), end in zip(order, ends):
            st = torch.cuda.Stream()
            with torch.cuda.stream(st):
                sim.run(0, steps)
                end.record(st)
        torch.cuda.synchronize()
        assert ends[0].elapsed_time(ends[1]) > 0.0
        assert fifo.counters()["error_bits"] == 0 and ring.counters()["error_bits"] == 0
    ref = oracle.Run(small, oracle.RING, 0, n_steps=1000, n_threads=8)
    np.testing.assert_array_equal(ring.tape()["U"].cpu().numpy().view(np.uint32), ref.U.view(np.uint32))
    ring.close()
    fifo.close()
