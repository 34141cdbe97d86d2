"""GPU tests of feed-forward networks on the MFMA path, which run several
ticks per launch (kern_mfma_ticks.hip): every core shape the form takes,
against the oracle element by element (output-bus spikes, potentials,
counters), with ragged sample counts, calls longer than a segment and calls of
one tick, axons of many sources, graph replays among eager, state-resident and
link-counting calls on one handle, and a workspace sized for the tick-by-tick
layout."""
import ctypes

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


def forward_net(seed, C, A, N, G, b, gw, reach=3, axons=None, **extra):
    """A random network whose spikes only ever go to a core of a higher index
    (at most `reach` on); axons: destination axons drawn from that many (few:
    many sources per axon)."""
    net = W.random_net(seed, C, A, N, G, weight_bits=b, grid_w=gw, density=0.25, p_core=0.85, p_out=0.1,
                       config_id=871, input_cores=[0, C // 2], **extra)
    r = np.random.default_rng(seed)
    src = np.repeat(np.arange(C)[:, None], N, axis=1)
    dst = np.minimum(src + r.integers(1, reach + 1, size=(C, N)), C - 1)
    core = (net.dest_kind == W.DEST_CORE) & (src < C - 1)
    net.dest_kind[(net.dest_kind == W.DEST_CORE) & ~core] = W.DEST_OUT
    dx, dy = W.relative_offsets(src, dst, gw)
    net.dest_dx[:] = np.where(core, dx, 0)
    net.dest_dy[:] = np.where(core, dy, 0)
    if axons:
        net.dest_axon[:] = np.where(core, net.dest_axon % axons, 0)
    net.dest_axon[~core] = 0
    net.dest_delay[~core] = 0
    return net


def check(net, S, chunks, rt=None, modes=None, rate=0.15):
    import torch
    from paper_2404_16208_amd.ranc import RancNet
    T = sum(chunks)
    x = W.bernoulli_inputs(3, net, S, T, rate, config_id=871)
    ref = oracle_results(net, x, T, range(S))
    xd = torch.from_numpy(x.view(np.int32)).cuda()
    g = RancNet(net, S, rt or max(chunks), path="mfma", workspace_fill=0xA5)
    modes = modes or ["eager"] * len(chunks)
    t = 0
    got = {s: [] for s in range(S)}
    for k, mode in zip(chunks, modes):
        log(f"[forward] {net.name} S={S} ticks {t}..{t + k} {mode}")
        g.count_links(mode == "links")
        g.run(xd[:, t:t + k].contiguous(), k, graph=mode == "graph", resident=mode == "resident")
        t += k
        for s in sorted({0, S - 1}):
            got[s].append(g.spikes(s, t - k, t))
    for s in sorted({0, S - 1}):
        assert np.array_equal(np.concatenate(got[s]), ref[s]["events"]), s
    for s in range(S):
        assert_sample_equal(g, ref[s], s, T, what=net.name)
    g.close()


SHAPES = [(64, 64), (64, 128), (64, 256), (64, 512), (128, 64), (128, 128), (128, 256), (128, 512), (256, 64), (256, 128),
          (256, 256), (256, 512), (512, 64), (512, 128), (512, 256), (512, 512)]


@pytest.mark.parametrize("model", [False, True])
@pytest.mark.parametrize("bits", [8, 9])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "A%dN%d" % s)
def test_every_shape(shape, bits, model):
    A, N = shape
    extra = dict(potential_bits=14, floor_range=(-300, -1), linear_frac=0.5) if model else {}
    net = forward_net(A + N + bits, 6, A, N, 4, bits, 3, **extra)
    check(net, 67, [9, 2, 1, 9])


@pytest.mark.parametrize("S", [1, 64, 129])
@pytest.mark.parametrize("chunks", [[32], [40, 33, 1], [31, 64]])
def test_segments(S, chunks):
    check(forward_net(11, 8, 128, 128, 2, 9, 4, max_delay=15), S, chunks, rt=64)


def test_many_sources_per_axon():
    check(forward_net(12, 5, 256, 256, 4, 9, 5, axons=24), 65, [17, 17], rate=0.3)


def test_levels_without_routing():
    net = forward_net(13, 4, 128, 128, 4, 8, 2)
    net.dest_kind[net.dest_kind == W.DEST_CORE] = W.DEST_OUT
    for f in (net.dest_dx, net.dest_dy, net.dest_axon, net.dest_delay):
        f[:] = 0
    check(net, 64, [16, 5])


def test_wide_levels():
    """Enough cores per level that the levels run one after another."""
    net = forward_net(14, 320, 64, 128, 2, 6, 20, reach=160)
    check(net, 64, [8, 8])


def test_calls_mixed_on_one_handle():
    net = forward_net(15, 6, 256, 256, 4, 9, 3)
    check(net, 70, [12] * 8, modes=["graph", "eager", "links", "graph", "resident", "graph", "links", "eager"])


def test_graph_replays():
    import torch
    from paper_2404_16208_amd.ranc import RancNet
    net = forward_net(16, 7, 256, 256, 4, 9, 7)
    S, k, calls = 66, 10, 5
    x = W.bernoulli_inputs(3, net, S, k * calls, 0.2, config_id=871)
    ref = oracle_results(net, x, k * calls, range(S))
    g = RancNet(net, S, k, path="mfma")
    buf = torch.empty((S, k) + x.shape[2:], dtype=torch.int32, device="cuda")
    got = []
    for i in range(calls):
        buf.copy_(torch.from_numpy(np.ascontiguousarray(x[:, i * k:(i + 1) * k]).view(np.int32)))
        g.run(buf, k, graph=True)
        got.append(g.spikes(S - 1, i * k, (i + 1) * k))
        (torch.ones(1 << 20, device="cuda") * 2).sum().item()   # the program's own work between replays
    assert np.array_equal(np.concatenate(got), ref[S - 1]["events"])
    for s in range(S):
        assert_sample_equal(g, ref[s], s, k * calls, what="replays")


def test_workspace_of_the_tick_by_tick_layout():
    """A workspace too small for the longer history ring but large enough for
    the tick-by-tick layout still loads; one page less does not."""
    import torch
    from paper_2404_16208_amd import ranc as R
    net = forward_net(17, 4, 256, 256, 4, 9, 2)
    S, T = 64, 16
    d = R.Desc(net)
    need = R.ranc_workspace_bytes(d, S, T, R.RANC_PATH_MFMA)
    slot = 4 * 256 * 8
    small = need - (T - 1) * slot - 256   # ring of D + 1 slots, no core order
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    st = torch.cuda.current_stream().cuda_stream
    h = ctypes.c_void_p(0)
    assert R._lib.ranc_load_network(ctypes.byref(d.c), S, T, R.RANC_PATH_MFMA, ws.data_ptr(), small - 256, st,
                                    ctypes.byref(h)) == R.RANC_ENOMEM
    x = W.bernoulli_inputs(3, net, S, T, 0.2, config_id=871)
    ref = oracle_results(net, x, T, [0, 63])
    xd = torch.from_numpy(x.view(np.int32)).cuda()
    for size in (small, need):
        handle = R.ranc_load_network(d, S, T, R.RANC_PATH_MFMA, ws.data_ptr(), size, st)
        R.ranc_run_ticks([handle], [xd.data_ptr()], R.RANC_INPUTS_ON_DEVICE, T, st)
        for s in (0, 63):
            assert np.array_equal(R.ranc_read_potentials(handle, s, 4, 256), ref[s]["v"]), (size, s)
            for k, v in R.ranc_read_counters(handle, s).items():
                assert v == ref[s]["counters"][k], (size, s, k)
        R.ranc_free(handle)
