"""Dense windows of the ring (role_dense: events summed in LDS tiles of all targets) against the oracle: trace bit for bit and
counters, in runs that change between dense and staged windows; tiles of the whole window and of a few rows, trial
boundaries inside a spike word, several window lengths; and long lists of spikes that were no candidates in the forward
kernel."""
import numpy as np
import pytest
import torch

from oracle import oracle
from paper_2512_05906_amd import adseq, synth

pytestmark = pytest.mark.gpu


def _went_dense(sim):
    """Whether the last window was (and the next one will be) expanded the dense way: Counters::dense, at byte 76 of the
    workspace, which begins with the counters."""
    base = -sim.workspace.data_ptr() % 256
    return sim.workspace[base + 76:base + 84].cpu().numpy().view(np.uint32).tolist()


@pytest.mark.parametrize("dense", ["1", "0"])
@pytest.mark.parametrize("n,b,fan,d_max,T,window,blocks", [(2000, 1, 100, 40, 130, 16, 16), (1501, 2, 90, 33, 110, 16, 16),
                                                           (6001, 1, 60, 50, 100, 16, 32), (900, 3, 120, 70, 200, 16, 32),
                                                           (500, 1, 120, 70, 200, 64, 8), (6000, 1, 80, 20, 60, 8, 16)])
def test_dense_windows(n, b, fan, d_max, T, window, blocks, dense, monkeypatch):
    monkeypatch.setenv("ADSEQ_RING_DENSE", dense)
    monkeypatch.setenv("ADSEQ_RING_WINDOW", str(window))
    monkeypatch.setenv("ADSEQ_RING_BINBLOCKS", str(blocks))
    wl = synth.ragged_network(n, fan, d_max, seed=n, rate_hz=2500.0, t=T, b=b, w_mean=1.2 / fan, w_std=1.0 / fan)
    ref = oracle.Run(wl, oracle.RING, 0, n_steps=T, batch=b, n_threads=8)
    per_step = ref.spikes.reshape(T, -1).sum(axis=1)
    recent = np.convolve(per_step, np.ones(d_max))[:T]
    assert recent.max() > 768 * blocks   # (windows with more row pieces than the blocks' queues hold)
    sim = adseq.Adseq(wl, adseq.RING, 0, batch=b, record_tape=True, max_steps=T, step_event_capacity=4000000)
    for _ in range(2):
        sim.run(0, T // 3); sim.step(T // 3); sim.run(T // 3 + 1, T - T // 3 - 1)
        torch.cuda.synchronize()
        np.testing.assert_array_equal(sim.tape()["U"].cpu().numpy().view(np.uint32), ref.U.view(np.uint32))
        c, rc = sim.counters(), ref.counters()
        for key in ("enqueued", "dropped", "delivered", "sum_enqueued", "sum_dropped", "sum_delivered"):
            assert c[key] == rc[key], key
        assert any(_went_dense(sim)) == (dense == "1")
        sim.reset()
    sim.close()
