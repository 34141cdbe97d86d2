"""GPU test of a single call long enough for its counts to pass 32 bits."""
import numpy as np
import pytest

from paper_2404_16208_amd import workloads as W

pytestmark = pytest.mark.gpu


def test_counts_of_a_call_past_32_bits():
    """One core whose 256 neurons fire on every tick, neuron i into axon i, all
    axons connected: from the second tick on 256 spikes are delivered and 64 *
    256 events counted per 64-neuron block and tick, 2^32 of them after 2^18
    ticks of one call. The potentials stay at their reset."""
    import torch
    from paper_2404_16208_amd.ranc import RancNet
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    N, T = 256, (1 << 18) + 100
    net = W.random_net(5, 1, N, N, 1, density=1.0, p_core=1.0, p_out=0.0, max_delay=1, leak_range=(9, 9), thr_range=(1, 1),
                       weight_range=(0, 0), reset_range=(-3, -3), input_cores=[], config_id=873)
    net.dest_axon[:] = np.arange(N)
    g = RancNet(net, 2, T, path="plain")
    g.run(None, T)
    for s in range(2):
        c = g.counters(s)
        assert c["emitted"] == c["routed"] == N * T and c["out"] == 0, s
        assert c["delivered"] == N * (T - 1) and c["events"] == N * N * (T - 1), s
        assert (g.potentials(s) == -3).all(), s
    g.close()
