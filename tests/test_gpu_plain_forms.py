"""GPU tests of the plain path's forms without a router: one launch per tick
(axons in natural order, or sorted by type), several samples per workgroup, a
block of ticks of a feed-forward network per launch, and a small network's
whole call in one launch; every output spike, potential and counter of every
sample against the oracle. Calls of every form follow each other on one handle
(the byte ring hands its scheduled spikes to the bit ring of the router and of
batches and back), with graph replays, link counting, one-tick calls, delays
up to 15 and a workspace sized for the layout without the byte ring."""
import ctypes

import numpy as np
import pytest

from paper_2404_16208_amd import workloads as W
from tests.parity_utils import assert_sample_equal, log, oracle_results
from tests.test_gpu_feedforward import forward_net

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2404_16208_amd import ranc  # noqa: F401


def check(net, S, chunks, modes=None, rate=0.2, inputs=True):
    """modes: "eager", "graph", "links", "router" (one lane per word), "batch"
    (with another network)."""
    import torch
    from paper_2404_16208_amd.ranc import RancNet, run_batch
    T = sum(chunks)
    x = W.bernoulli_inputs(3, net, S, T, rate, config_id=872) if inputs else None
    ref = oracle_results(net, x, T, range(S))
    xd = torch.from_numpy(x.view(np.int32)).cuda() if inputs else None
    g = RancNet(net, S, max(chunks), path="plain", workspace_fill=0xA5)
    other = W.random_net(9, 3, 64, 64, 2, grid_w=3, config_id=872)
    auto = g.launch_shape()
    t = 0
    got = []
    for k, mode in zip(chunks, modes or ["eager"] * len(chunks)):
        log(f"[plain] {net.name} S={S} ticks {t}..{t + k} {mode}")
        g.count_links(mode == "links")
        g.launch_shape(dict(auto, route_lanes_per_word=1) if mode == "router" else auto)
        xi = xd[:, t:t + k].contiguous() if inputs else None
        if mode == "batch":
            run_batch([g, RancNet(other, 2, k, path="plain")], [xi, None], k)
        else:
            g.run(xi, k, graph=mode == "graph")
        t += k
        got.append(g.spikes(S - 1, t - k, t))
    assert np.array_equal(np.concatenate(got), ref[S - 1]["events"])
    for s in range(S):
        assert_sample_equal(g, ref[s], s, T, what=net.name)
    g.close()


def recurrent(seed, C, A, N, G, gw, **kw):
    return W.random_net(seed, C, A, N, G, grid_w=gw, density=0.25, p_core=0.85, p_out=0.1, config_id=872,
                        input_cores=list(range(0, C, 2)), **kw)


SHAPES = [(A, N) for A in (64, 128, 256, 512) for N in (64, 128, 256, 512)]


@pytest.mark.parametrize("G", [1, 2, 4, 8])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "A%dN%d" % s)
def test_shapes_one_launch_per_tick_and_whole_call(shape, G):
    """Short calls run one launch per tick; the long one the whole network in
    one launch where it fits (at most 4096 neurons)."""
    A, N = shape
    model = dict(potential_bits=14, floor_range=(-300, -1), linear_frac=0.5) if (A + G) % 3 == 0 else {}
    check(recurrent(A + N + G, 6, A, N, G, 3, max_delay=1 + (A // 64 + G) % 15, **model), 3, [1, 3, 34, 2])


@pytest.mark.parametrize("C", [1, 5, 12, 16])
def test_whole_call_sizes(C):
    check(recurrent(40 + C, C, 256, 256, 4, C, max_delay=15), 2, [12, 13, 40])


@pytest.mark.parametrize("types", ["one", "two_uneven"])
def test_uneven_types(types):
    net = recurrent(50, 4, 256, 256, 4, 2)
    net.axon_type[:] = 0 if types == "one" else (np.arange(256) < 250).astype(np.uint8)
    check(net, 2, [5, 20])


def test_without_input_and_output():
    net = W.random_net(51, 4, 64, 128, 2, max_delay=2, grid_w=2, p_core=1.0, p_out=0.0, leak_range=(5, 20),
                       thr_range=(10, 40), input_cores=[], config_id=872)
    check(net, 3, [3, 20], inputs=False)


@pytest.mark.parametrize("S", [1, 33])
def test_sorted_and_several_samples_per_workgroup(S):
    # 300 cores: past 2^18 neuron-samples the columns are sorted by type, and
    # 33 samples take several per workgroup
    check(recurrent(52, 300 if S > 1 else 1024, 64, 256, 4, 20 if S > 1 else 32), S, [4, 3])


@pytest.mark.parametrize("shape", [(64, 64), (128, 256), (256, 256), (512, 128)], ids=lambda s: "A%dN%d" % s)
@pytest.mark.parametrize("S", [1, 5])
def test_feed_forward_blocks(shape, S):
    A, N = shape
    check(forward_net(A + N, 30, A, N, 4, 9, 6, max_delay=7), S, [32, 1, 40, 9], modes=["eager", "graph", "graph", "eager"])


def test_feed_forward_forms_mixed():
    check(forward_net(60, 24, 128, 128, 2, 8, 6, axons=16), 3, [11] * 8,
          modes=["eager", "router", "graph", "batch", "links", "graph", "batch", "eager"])


@pytest.mark.parametrize("C", [6, 40])
def test_forms_mixed(C):
    check(recurrent(61, C, 128, 128, 4, 2, max_delay=9), 3, [13] * 9,
          modes=["graph", "router", "eager", "batch", "links", "graph", "router", "graph", "batch"])


def test_graph_replays():
    import torch
    from paper_2404_16208_amd.ranc import RancNet
    for C, k in ((6, 14), (60, 6)):
        net = recurrent(62, C, 128, 256, 4, 3)
        S, calls = 2, 5
        x = W.bernoulli_inputs(3, net, S, k * calls, 0.2, config_id=872)
        ref = oracle_results(net, x, k * calls, range(S))
        g = RancNet(net, S, k, path="plain")
        buf = torch.empty((S, k) + x.shape[2:], dtype=torch.int32, device="cuda")
        got = []
        for i in range(calls):
            buf.copy_(torch.from_numpy(np.ascontiguousarray(x[:, i * k:(i + 1) * k]).view(np.int32)))
            g.run(buf, k, graph=True)
            got.append(g.spikes(1, i * k, (i + 1) * k))
            (torch.ones(1 << 20, device="cuda") * 2).sum().item()   # the program's own work between replays
        assert np.array_equal(np.concatenate(got), ref[1]["events"])
        for s in range(S):
            assert_sample_equal(g, ref[s], s, k * calls, what=f"replays C{C}")


def test_workspace_without_the_byte_ring():
    """A workspace that holds everything but the byte ring still loads (and
    runs through the router)."""
    import torch
    from paper_2404_16208_amd import ranc as R
    net = recurrent(63, 8, 256, 256, 4, 4)
    S, T = 3, 6
    d = R.Desc(net)
    need = R.ranc_workspace_bytes(d, S, T, R.RANC_PATH_PLAIN)
    small = need - (4 + 2) * S * 8 * 256   # the byte ring alone (max_delay 4)
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    st = torch.cuda.current_stream().cuda_stream
    x = W.bernoulli_inputs(3, net, S, T, 0.2, config_id=872)
    ref = oracle_results(net, x, T, range(S))
    xd = torch.from_numpy(x.view(np.int32)).cuda()
    h = ctypes.c_void_p(0)
    assert R._lib.ranc_load_network(ctypes.byref(d.c), S, T, R.RANC_PATH_PLAIN, ws.data_ptr(), need // 4, st,
                                    ctypes.byref(h)) == R.RANC_ENOMEM
    for size in (small, need):
        handle = R.ranc_load_network(d, S, T, R.RANC_PATH_PLAIN, ws.data_ptr(), size, st)
        R.ranc_run_ticks([handle], [xd.data_ptr()], R.RANC_INPUTS_ON_DEVICE, T, st)
        for s in range(S):
            assert np.array_equal(R.ranc_read_potentials(handle, s, 8, 256), ref[s]["v"]), (size, s)
            for k, v in R.ranc_read_counters(handle, s).items():
                assert v == ref[s]["counters"][k], (size, s, k)
        R.ranc_free(handle)


@pytest.mark.parametrize("graph", [False, True])
def test_batch_of_every_form(graph):
    """One batch of networks that run one launch per tick on the byte ring
    (every core shape of the wave form), a whole call in one launch, blocks of
    ticks on both paths, and the MFMA tick loop; called twice."""
    import torch
    from paper_2404_16208_amd.ranc import RancNet, run_batch
    T = 14
    nets = [(recurrent(70 + i, 5, A, N, G, 5, max_delay=1 + i), "plain", 9) for i, (A, N, G) in
            enumerate([(64, 512, 1), (512, 64, 8), (128, 128, 2), (256, 256, 4), (512, 512, 8)])]
    nets += [(recurrent(80, 40, 128, 128, 4, 8), "plain", 7), (recurrent(81, 24, 256, 64, 2, 6, potential_bits=12), "plain", 5),
             (forward_net(82, 30, 128, 128, 4, 8, 6), "plain", 3), (forward_net(83, 6, 256, 256, 4, 9, 3), "mfma", 70),
             (recurrent(84, 6, 256, 128, 4, 3), "mfma", 65)]
    gs, xs, refs = [], [], []
    for net, path, S in nets:
        x = W.bernoulli_inputs(3, net, S, 2 * T, 0.2, config_id=872)
        refs.append(oracle_results(net, x, 2 * T, sorted({0, S - 1})))
        xs.append(torch.from_numpy(x.view(np.int32)).cuda())
        gs.append(RancNet(net, S, T, path=path, workspace_fill=0xA5))
    bufs = [torch.empty((x.shape[0], T) + tuple(x.shape[2:]), dtype=torch.int32, device="cuda") for x in xs]
    for call in range(2):
        for b, x in zip(bufs, xs):
            b.copy_(x[:, call * T:(call + 1) * T])
        run_batch(gs, bufs, T, graph=graph)
        torch.cuda.synchronize()
    for g, ref in zip(gs, refs):
        for s, r in ref.items():
            assert_sample_equal(g, r, s, 2 * T, what=f"{g.net.name}/{g.path}")


@pytest.mark.parametrize("persistent", [False, True])
@pytest.mark.parametrize("links", [False, True])
def test_batch_of_networks_with_launches_of_their_own(links, persistent):
    """Plain networks from 2^17 neurons times samples on (one just below, one
    with the router asked for) beside small ones, over three calls."""
    import torch
    from paper_2404_16208_amd.ranc import RancNet, run_batch
    T = 5
    nets = [(recurrent(90, 64, 128, 128, 4, 8), 16), (recurrent(91, 32, 256, 128, 2, 8, potential_bits=12), 31),
            (recurrent(92, 100, 64, 64, 8, 10, max_delay=9), 21), (recurrent(93, 24, 512, 256, 4, 6), 23),
            (recurrent(94, 4, 64, 64, 1, 2), 3)]
    gs, xs, refs = [], [], []
    for i, (net, S) in enumerate(nets):
        x = W.bernoulli_inputs(3, net, S, 3 * T, 0.2, config_id=872)
        refs.append(oracle_results(net, x, 3 * T, [0, S - 1]))
        xs.append(torch.from_numpy(x.view(np.int32)).cuda())
        g = RancNet(net, S, T, path="plain", workspace_fill=0xA5)
        g.count_links(links and i % 2 == 0)
        if i == 3:
            g.launch_shape(dict(g.launch_shape(), route_lanes_per_word=1))
        gs.append(g)
    for call in range(3):
        run_batch(gs, [x[:, call * T:(call + 1) * T].contiguous() for x in xs], T, graph=call > 0, persistent=persistent)
    for (net, S), g, ref in zip(nets, gs, refs):
        for s, r in ref.items():
            assert_sample_equal(g, r, s, 3 * T, what=f"{net.name} links={links}")


# (cores, samples): below, at and above the million neurons times samples and
# the 32 samples from which RANC_PATH_AUTO takes the MFMA path
@pytest.mark.parametrize("C,S,path", [(128, 31, "plain"), (128, 32, "mfma"), (127, 32, "plain"), (66, 63, "mfma")])
def test_automatic_path_below_64_samples(C, S, path):
    """Results against the oracle and the plain path's, what the handle
    accepts, and the plain path in a workspace sized for it."""
    import torch
    from paper_2404_16208_amd import ranc as R
    net = recurrent(95, C, 256, 256, 4, C if C == 127 else C // 2)
    T = 6
    x = W.bernoulli_inputs(3, net, S, T, 0.2, config_id=872)
    ref = oracle_results(net, x, T, [0, S - 1])
    xd = torch.from_numpy(x.view(np.int32)).cuda()
    for which in ("auto", "plain"):
        g = R.RancNet(net, S, T, path=which, workspace_fill=0xA5)
        assert g.path == (path if which == "auto" else "plain")
        router = dict(samples_per_wg=0, route_samples_per_block=1, route_split=2, route_stage=0, route_lanes_per_word=1)
        g.launch_shape(router)
        with pytest.raises(R.RancError):
            g.launch_shape(dict(router, route_split=0))
        with pytest.raises(R.RancError):
            g.run(xd, T, resident=True)
        g.run(xd[:, :2].contiguous(), 2)
        R.run_batch([g, R.RancNet(net, 2, 4, path="plain")], [xd[:, 2:].contiguous(), xd[:2, 2:].contiguous()], T - 2)
        for s, r in ref.items():
            assert_sample_equal(g, r, s, T, what=which)
        g.close()
    d = R.Desc(net)
    size = R.ranc_workspace_bytes(d, S, T, R.RANC_PATH_PLAIN)
    ws = torch.empty(size, dtype=torch.uint8, device="cuda")
    st = torch.cuda.current_stream().cuda_stream
    h = R.ranc_load_network(d, S, T, R.RANC_PATH_AUTO, ws.data_ptr(), size, st)
    R.ranc_run_ticks([h], [xd.data_ptr()], R.RANC_INPUTS_ON_DEVICE, T, st)
    for s, r in ref.items():
        assert np.array_equal(R.ranc_read_potentials(h, s, C, 256), r["v"])
    R.ranc_free(h)
