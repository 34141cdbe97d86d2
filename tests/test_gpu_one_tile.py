"""GPU tests of the MFMA path's form for workgroups of one 64-sample tile: every
core shape and plane count with the B tiles read from the int8 planes and built
from the compact crossbar, sample counts at the edges of groups and tiles, axons
with several sources, both potential updates, alone and in a batch; every output
spike, potential and counter against the oracle."""
import numpy as np
import pytest

from paper_2404_16208_amd import workloads as W
from tests.parity_utils import assert_sample_equal, log, oracle_results

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2404_16208_amd import ranc  # noqa: F401


# samples: one, the edges of a 32-sample group and of a tile, two tiles
@pytest.mark.parametrize("S", [1, 32, 33, 64, 100])
@pytest.mark.parametrize("bsrc", ["planes", "compact"])
@pytest.mark.parametrize("A", [64, 128, 256, 512])
def test_one_tile_shapes(A, bsrc, S, monkeypatch):
    import torch
    from paper_2404_16208_amd.ranc import RancNet, run_batch
    monkeypatch.setenv("RANC_MFMA_BSRC", bsrc)
    monkeypatch.setenv("RANC_MFMA_SPW", "64")
    T = 5
    gs, xs, refs = [], [], []
    for i, (N, bits) in enumerate((N, bits) for N in (64, 128, 256, 512) for bits in (8, 9)):
        kw = dict(potential_bits=13) if i % 3 == 1 else {}
        net = W.random_net(500 + i, 4, A, N, (2, 8)[i % 2], grid_w=2, density=0.3, p_core=0.8, p_out=0.15,
                           max_delay=1 + i % 3, weight_bits=bits, input_cores=[0, 3], config_id=880, **kw)
        x = W.bernoulli_inputs(3, net, S, 2 * T, 0.25, config_id=880)
        log(f"[one tile] A{A} N{N} bits{bits} S{S} {bsrc}")
        refs.append(oracle_results(net, x, 2 * T, sorted({0, S // 2, S - 1})))
        xs.append(torch.from_numpy(x.view(np.int32)).cuda())
        g = RancNet(net, S, T, path="mfma", workspace_fill=0xA5)
        assert g.launch_shape()["samples_per_wg"] == 64
        gs.append(g)
    for g, x in zip(gs, xs):
        g.run(x[:, :T].contiguous(), T)
    run_batch(gs, [x[:, T:].contiguous() for x in xs], T)
    for g, ref in zip(gs, refs):
        for s, r in ref.items():
            assert_sample_equal(g, r, s, 2 * T, what=g.net.name)
        g.close()


@pytest.mark.parametrize("S", [8, 9, 31, 32, 33])
def test_event_driven_partial_tiles(S):
    """The event-driven path's potentials of valid samples only (up to 32 samples)
    and of whole tiles, both potential updates."""
    import torch
    from paper_2404_16208_amd.ranc import RancNet
    T = 6
    for i, kw in enumerate((dict(), dict(potential_bits=13))):
        net = W.random_net(540 + i, 6, 128, 256 if i else 64, 4, grid_w=3, density=0.3, p_core=0.8, p_out=0.15,
                           max_delay=3, input_cores=[0, 3], config_id=881, **kw)
        x = W.bernoulli_inputs(3, net, S, T, 0.25, config_id=881)
        ref = oracle_results(net, x, T, range(S))
        g = RancNet(net, S, T, path="sparse", workspace_fill=0xA5)
        xd = torch.from_numpy(x.view(np.int32)).cuda()
        g.run(xd[:, :2].contiguous(), 2)
        g.run(xd[:, 2:].contiguous(), T - 2)
        for s in range(S):
            assert_sample_equal(g, ref[s], s, T, what=f"event S{S}")
        g.close()
