"""The resident step kernels of the ring with synaptic current states and with state arrays that are no multiple of
four cells (ring_resident_forward.h, ring_flow_reverse.h), against the oracle and against one launch per step: trace bit
for bit, gradients, both gradient modes; one, four and eight neurons per thread, one block and many."""
import numpy as np
import pytest
import torch

from oracle import oracle
from paper_2512_05906_amd import adseq, synth
from tests import helpers as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("surrogate", [adseq.SURR_SUPERSPIKE, adseq.GRAD_SPIKE_TIME])
@pytest.mark.parametrize("n,b,T,tau_syn,tau_rise,continuous,blocks", [
    (701, 3, 90, 5.0, 0.0, False, ""), (3001, 1, 70, 2.0, 0.0, True, ""), (12004, 2, 50, 5.0, 0.0, False, "16"),
    (20004, 1, 40, 5.0, 0.0, False, "8"), (2501, 1, 70, 5.0, 1.0, False, ""), (257, 1, 60, 0.0, 0.0, False, ""),
    (43690, 3, 34, 0.0, 0.0, False, "")])
def test_resident_states_and_odd_sizes(surrogate, n, b, T, tau_syn, tau_rise, continuous, blocks, monkeypatch):
    monkeypatch.setenv("ADSEQ_RING_REVERSE_WINDOWS", "0")
    if blocks:   # (few blocks: four and eight neurons per thread)
        monkeypatch.setenv("ADSEQ_RING_REVERSE_BLOCKS", blocks)
        monkeypatch.setenv("ADSEQ_RING_FORWARD_BLOCKS", blocks)
    wl = synth.ragged_network(n, 60, 30, seed=n, rate_hz=500.0, t=T, b=b, w_mean=0.01, w_std=0.01, continuous=continuous)
    wl.tau_syn_ms, wl.tau_rise_ms = tau_syn, tau_rise
    ref = oracle.Run(wl, oracle.RING, 0, n_steps=T, batch=b, surrogate=surrogate, n_threads=8)
    assert ref.spikes.sum() > 50
    rng = np.random.default_rng(n)
    dc = rng.normal(0, 1e-3, (b, n)).astype(np.float32)
    dU = rng.normal(0, 1e-4, (T, b, n)).astype(np.float32)
    gw, gd = ref.backward(dc, dU)
    for resident in ("1", "0"):
        monkeypatch.setenv("ADSEQ_RING_FORWARD_CHIP", resident)
        monkeypatch.setenv("ADSEQ_RING_RESIDENT", "0")
        monkeypatch.setenv("ADSEQ_RING_RESIDENT_REVERSE", resident)
        sim = adseq.Adseq(wl, adseq.RING, 0, batch=b, record_tape=True, max_steps=T, surrogate=surrogate)
        sim.profile(True)
        sim.run(0, 19); sim.step(19); sim.run(20, T - 20)
        g_w, g_d = (torch.empty(wl.n_synapses, device=sim.dev) for _ in range(2))
        sim.backward(torch.from_numpy(dc).to(sim.dev), torch.from_numpy(dU).to(sim.dev), g_w, g_d)
        torch.cuda.synchronize()
        p = sim.profile_read()
        assert (p["lif"]["launches"] < T) == (resident == "1")
        assert (p["bwd_neurons"]["launches"] < T) == (resident == "1" and tau_rise == 0.0)
        np.testing.assert_array_equal(sim.tape()["U"].cpu().numpy().view(np.uint32), ref.U.view(np.uint32))
        assert sim.counters()["error_bits"] == 0 and sim.counters()["delivered"] == ref.counters()["delivered"]
        H.grad_close(g_w.cpu().numpy(), gw)
        H.grad_close(g_d.cpu().numpy(), gd)
        sim.close()
