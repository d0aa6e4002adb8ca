"""Gradients on their way to the host: every part arrives, from the call's own inputs, on any
stream and from several contexts and threads at a time."""
import threading

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

NORM = dict(in_shift=[0.0] * 4, in_scale=[1.0] * 4, out_scale=[1.0] * 4, lrr_scale=1.0)


def context(H, W, B, seed):
    from paper_1812_00118_amd.surrogate import Surrogate, init_params
    sur = Surrogate(H, W, B, NORM)
    sur.set_params(init_params(seed))
    g = torch.Generator(device="cuda").manual_seed(seed)
    return sur, [(torch.randn((B, H, W, 8), generator=g, device="cuda").to(torch.bfloat16),
                  torch.randn((B, H, W, 4), generator=g, device="cuda")) for _ in range(2)]


@pytest.mark.parametrize("shape", [(16, 16, 1), (64, 48, 3)], ids=str)
def test_gradients_of_streams_and_threads_are_the_same(shape):
    sets = [context(*shape, seed) for seed in (1, 2)]
    want = [[sur.gradients(x, y) for x, y in batches] for sur, batches in sets]
    for w in want:
        assert all(np.all(np.isfinite(g)) and np.isfinite(loss) for g, loss in w)
        assert not np.array_equal(w[0][0], w[1][0])
    torch.cuda.synchronize()
    got = [[] for _ in sets]

    def work(k):
        sur, batches = sets[k]
        for _ in range(4):
            with torch.cuda.stream(torch.cuda.Stream()):
                got[k].append([sur.gradients(x, y) for x, y in batches])

    threads = [threading.Thread(target=work, args=(k,)) for k in range(len(sets))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for w, runs in zip(want, got):
        assert len(runs) == 4
        for run in runs:
            for (g, loss), (g2, loss2) in zip(w, run):
                assert np.array_equal(g, g2) and loss == loss2
