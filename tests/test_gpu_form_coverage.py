"""GPU tests of the forms that run several ticks per launch, on networks for which
the cost model takes them (each call's launches are counted, so a changed model
cannot empty a test): every core shape, plane count, neuron model and source
count of the MFMA form, every shape, type count and axon order of the plain
block form, skewed and wide levels, uneven axon types; output-bus spikes,
potentials and counters against the oracle."""
import numpy as np
import pytest

from paper_2404_16208_amd import workloads as W
from tests.parity_utils import assert_sample_equal, log, oracle_results

pytestmark = pytest.mark.gpu

MODEL = dict(potential_bits=14, floor_range=(-300, -1), linear_frac=0.5)
SHAPES = [(A, N) for A in (64, 128, 256, 512) for N in (64, 128, 256, 512)]


def layers_net(seed, levels, per, A, N, G, bits=9, several=True, skip=False, **kw):
    """`levels` layers of `per` cores: neurons send to the next layer (skip: to any
    later one), to any axon (several sources per axon) or each axon from one
    neuron at most; the last layer's and every twentieth neuron go to the output
    bus. External input to the first layer and one core of the last."""
    C = levels * per
    net = W.random_net(seed, C, A, N, G, weight_bits=bits, grid_w=per, density=0.25, p_core=0.0, p_out=0.0, config_id=874,
                       input_cores=list(range(per)) + [C - 1], **kw)
    r = np.random.default_rng(seed)
    src = np.repeat(np.arange(C)[:, None], N, axis=1)
    if several:
        slot = r.integers(0, per * A, size=(C, N))
    else:
        slot = np.concatenate([r.permutation(per * max(A, N))[:per * N] for _ in range(levels)]).reshape(C, N)
    level = src // per + (r.integers(1, levels, size=(C, N)) if skip else 1)
    core = (level < levels) & (slot < per * A) & (np.arange(N) % 20 != 19)
    dst = np.where(core, level * per + slot // A, src)
    net.dest_kind[:] = np.where(core, W.DEST_CORE, np.where(np.arange(N) % 20 == 7, W.DEST_NONE, W.DEST_OUT))
    dx, dy = W.relative_offsets(src, dst, per)
    net.dest_dx[:], net.dest_dy[:] = np.where(core, dx, 0), np.where(core, dy, 0)
    net.dest_axon[:] = np.where(core, slot % A, 0)
    net.dest_delay[:] = np.where(core, r.integers(1, net.max_delay + 1, size=(C, N)), 0)
    return net


def check(net, path, S, calls, rt=None, samples=None, rate=0.2):
    """calls: (ticks, whether they take fewer launches of the integration than ticks)."""
    import torch
    from paper_2404_16208_amd.ranc import RancNet
    T = sum(k for k, _ in calls)
    x = W.bernoulli_inputs(3, net, S, T, rate, config_id=874)
    samples = range(S) if samples is None else samples
    ref = oracle_results(net, x, T, samples)
    xd = torch.from_numpy(x.view(np.int32)).cuda()
    g = RancNet(net, S, rt or max(k for k, _ in calls), path=path, workspace_fill=0xA5)
    t, last = 0, samples[-1]
    got = []
    for k, several in calls:
        log(f"[form] {path} C{net.num_cores}A{net.num_axons}N{net.num_neurons}G{net.num_types}b{net.weight_bits} S={S} ticks {t}..{t + k}")
        g.profile(True).run(xd[:, t:t + k].contiguous(), k)
        launches = g.profile_read()["integrate_launches"]
        assert 0 < launches < k if several else launches == k
        t += k
        got.append(g.spikes(last, t - k, t))
    assert np.array_equal(np.concatenate(got), ref[last]["events"])
    for s in samples:
        assert_sample_equal(g, ref[s], s, T, what=path)
    assert ref[last]["counters"]["delivered"] > 0
    g.close()


@pytest.mark.parametrize("bits", [8, 9])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "A%dN%d" % s)
def test_mfma_blocks_of_every_shape(shape, bits):
    A, N = shape
    several_ticks = A * (bits - 7) <= 512   # (512 axons with two planes run tick by tick)
    for i, (several, model) in enumerate([(False, {}), (True, {}), (False, MODEL), (True, MODEL)]):
        net = layers_net(A + N + i, 2, 2, A, N, 4, bits, several, max_delay=3 + 4 * i, **model)
        check(net, "mfma", 67, [(12, several_ticks), (1, False), (9, several_ticks)], samples=[0, 31, 32, 64, 66])


def test_mfma_skewed_levels():
    check(layers_net(1, 4, 3, 128, 256, 4, skip=True, max_delay=15), "mfma", 33, [(32, True), (1, False), (40, True), (32, True)], rt=64)


def test_mfma_wide_levels():
    check(layers_net(2, 3, 160, 64, 64, 2, 6), "mfma", 64, [(16, True), (16, True)], samples=[0, 63])


def uneven(net, most):
    """`most` of the axons of one type, the others spread over the rest (from four
    types on, but the last)."""
    G, i = net.num_types, np.arange(net.num_axons)
    others = [g for g in range(G) if g != G // 2 and (G < 4 or g < G - 1)] or [0]
    net.axon_type[:] = np.where(i < most, G // 2, np.array(others)[i % len(others)])
    return net


def plain_block_nets(A, N):
    """Networks of every type count above the whole-call form's size, their axons
    evenly of each type (columns sorted by type) and mostly of one (natural
    order where the sorted columns would be too many)."""
    per = 4096 // (2 * N) + 1
    for i, G in enumerate((1, 2, 4, 8)):
        for j in range(2):
            net = layers_net(A + N + i, 2, per, A, N, G, 6 + i, several=bool((i + j) % 2), max_delay=15 - 3 * i,
                             **(MODEL if (i + A // 64) % 2 else {}))
            yield uneven(net, A - 1) if j else net


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "A%dN%d" % s)
def test_plain_blocks_of_every_shape(shape):
    for net in plain_block_nets(*shape):
        check(net, "plain", 2, [(17, True), (1, False), (20, True)])


def test_plain_skewed_levels():
    check(layers_net(3, 4, 12, 128, 128, 4, skip=True, max_delay=9), "plain", 3, [(32, True), (1, False), (40, True), (32, True)], rt=64)


def large_natural_net(G):
    """Columns past what stays in cache: natural order for any type count."""
    return layers_net(4, 2, 1040, 64, 128, G, max_delay=2)


@pytest.mark.parametrize("G", [1, 2])
def test_plain_blocks_in_natural_order(G):
    check(large_natural_net(G), "plain", 1, [(9, True), (4, True)])


# (types, axons, most of one type): every word count per type that the sorted
# columns hold beyond the evenly spread types'
UNEVEN = [(2, 256, 190), (2, 256, 160), (2, 512, 256), (4, 256, 128), (4, 512, 192), (8, 256, 60), (8, 512, 96)]


@pytest.mark.parametrize("G,A,most", UNEVEN)
def test_uneven_types_in_sorted_order(G, A, most):
    """One launch per tick (enough work for the sorted columns), then the whole
    call in one launch where it fits."""
    net = uneven(W.random_net(G + A + most, 6, A, 256, G, grid_w=3, density=0.25, p_core=0.85, p_out=0.1, max_delay=6,
                              input_cores=[0, 3], config_id=874), most)
    whole = G * -(-most // 32) <= 12
    check(net, "plain", 171, [(5, False), (14, whole)], samples=[0, 1, 99, 170])


@pytest.mark.parametrize("D", [3, 7, 12], ids=["dmax4", "dmax8", "dmax16"])
@pytest.mark.parametrize("lanes", [1, 8])
def test_routers_without_the_byte_ring(D, lanes):
    """Both routers in a workspace that holds everything but the byte ring, with
    every delay-register width, launches and a graph."""
    import torch
    from paper_2404_16208_amd import ranc as R
    net = W.random_net(300 + D, 24, 128, 128, 4, max_delay=D, grid_w=6, density=0.25, p_core=0.85, p_out=0.1,
                       input_cores=list(range(0, 24, 3)), config_id=874)
    S, T = 5, D + 2
    d = R.Desc(net)
    small = R.ranc_workspace_bytes(d, S, T, R.RANC_PATH_PLAIN) - (D + 2) * S * 24 * 128
    ws = torch.full((small + 256,), 0xA5, dtype=torch.uint8, device="cuda")
    st = torch.cuda.current_stream().cuda_stream
    x = W.bernoulli_inputs(3, net, S, 2 * T, 0.25, config_id=874)
    ref = oracle_results(net, x, 2 * T, range(S))
    xd = torch.from_numpy(x.view(np.int32)).cuda()
    h = R.ranc_load_network(d, S, T, R.RANC_PATH_PLAIN, ws.data_ptr(), small, st)
    R.ranc_set_launch_shape(h, dict(R.ranc_get_launch_shape(h), route_lanes_per_word=lanes))
    for call in range(2):
        xi = xd[:, call * T:(call + 1) * T].contiguous()
        R.ranc_run_ticks([h], [xi.data_ptr()], R.RANC_INPUTS_ON_DEVICE | (R.RANC_RUN_GRAPH if call else 0), T, st)
        torch.cuda.synchronize()
    for s in range(S):
        assert np.array_equal(R.ranc_read_potentials(h, s, 24, 128), ref[s]["v"]), s
        for k, v in R.ranc_read_counters(h, s).items():
            assert v == ref[s]["counters"][k], (s, k)
    R.ranc_free(h)


def test_forms_among_replays_of_a_callers_graph():
    """Runs recorded into the caller's own graphs, without a router and with one,
    replayed among calls of the other form: every tick against the oracle."""
    import torch
    from paper_2404_16208_amd.ranc import RancNet
    net = W.random_net(31, 40, 128, 128, 4, max_delay=9, grid_w=8, density=0.25, p_core=0.85, p_out=0.1,
                       input_cores=list(range(0, 40, 3)), config_id=874)
    S, k = 3, 5
    plan = ["bytes", "record bytes", "words", "replay bytes", "words", "record words", "words", "replay words", "replay bytes",
            "bytes", "replay words", "replay words", "words", "bytes"]
    T = k * sum(not p.startswith("record") for p in plan)
    x = W.bernoulli_inputs(3, net, S, T, 0.2, config_id=874)
    ref = oracle_results(net, x, T, range(S))
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        g = RancNet(net, S, k, path="plain", workspace_fill=0xA5)
        auto = g.launch_shape()
        buf = torch.empty((S, k) + x.shape[2:], dtype=torch.int32, device="cuda")
        graphs, t = {}, 0
        for step in plan:
            log(f"[graphs] tick {t} {step}")
            what, form = step.split() if " " in step else ("run", step)
            if what != "replay":
                g.launch_shape(dict(auto, route_lanes_per_word=1 if form == "words" else 8))
            if what == "record":
                graphs[form] = torch.cuda.CUDAGraph()
                with torch.cuda.graph(graphs[form], stream=side):
                    g.run(buf, k)
                continue
            buf.copy_(torch.from_numpy(np.ascontiguousarray(x[:, t:t + k]).view(np.int32)))
            if what == "replay":
                graphs[form].replay()
            else:
                g.run(buf, k)
            t += k
        side.synchronize()
        for s in range(S):
            assert np.array_equal(g.potentials(s), ref[s]["v"]), s
            for c, v in g.counters(s).items():
                assert v == ref[s]["counters"][c], (s, c)
        g.close()


@pytest.mark.parametrize("case", ["whole", "ticks", "words", "blocks", "mfma_blocks", "mfma", "sparse"])
def test_reset_after_calls_of_every_form(case):
    """From the state that a call leaves (spikes scheduled up to 15 ticks ahead, at
    several ring positions) a reset gives the initial one."""
    import torch
    from paper_2404_16208_amd.ranc import RancNet
    path = "mfma" if case.startswith("mfma") else "sparse" if case == "sparse" else "plain"
    if case.endswith("blocks"):
        net = layers_net(7, 3, 8, 128, 256, 4, max_delay=15)
    else:
        net = W.random_net(32, 40 if case in ("ticks", "words") else 6, 128, 128, 4, max_delay=15, grid_w=2, density=0.25,
                           p_core=0.85, p_out=0.1, config_id=874)
    S, T = 70 if path != "plain" else 5, 19
    x = W.bernoulli_inputs(3, net, S, T, 0.2, config_id=874)
    ref = oracle_results(net, x, T, [0, S - 1])
    xd = torch.from_numpy(x.view(np.int32)).cuda()
    g = RancNet(net, S, T, path=path, workspace_fill=0xA5)
    if case == "words":
        g.launch_shape(dict(g.launch_shape(), route_lanes_per_word=1))
    for first in (0, 19, 13, 1):
        log(f"[reset] {case} after {first} ticks")
        if first:
            g.run(xd[:, :first].contiguous(), first, graph=first == 13)
        g.reset()
        g.run(xd, T)
        for s, r in ref.items():
            assert_sample_equal(g, r, s, T, what=f"{case} after {first}")
        g.reset()
    g.close()
