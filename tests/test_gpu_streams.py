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
