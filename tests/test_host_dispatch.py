"""What a call queues (kernels, streams, waits), by the built library's host code
on a HIP runtime that only keeps a log (dry_hip.py): no GPU."""
import os

import pytest

from paper_2404_16208_amd import build
from tests import dry_hip

pytestmark = pytest.mark.skipif(not os.path.exists(build.LIB), reason="needs the built library")


@pytest.fixture(scope="module")
def dry(tmp_path_factory):
    lib = dry_hip.build(tmp_path_factory.mktemp("dry"))
    return lambda body: dry_hip.run(lib, body)


@pytest.mark.parametrize("T,launches", [(65536, 1), (65537, 2), (200000, 4)])
def test_whole_call_form_in_bounded_launches(dry, T, launches):
    """The whole-call kernel sums its counts in 32 bits, for at most 2^16 ticks."""
    k = dry(f"""
net = W.random_net(1, 1, 64, 64, 1, input_cores=[], config_id=873)
result = kernels(run(load(net, 1, {T}, "plain"), {T}))
""")
    assert k == ["k_plain_whole"] * launches + ["k_advance_tick"]


def test_autotune_times_the_launches_that_the_shape_applies_to(dry):
    """A feed-forward network runs several ticks per launch whatever its samples
    per workgroup: the candidates (64 and 128 here) are timed tick by tick."""
    T = 16
    run, tuned, tune = dry(f"""
net = forward_net(17, 4, 256, 256, 4, 9, 2)
h = load(net, 128, {T}, "mfma")
result = [kernels(run(h, {T}))]
tune = R.ranc_autotune(h, 0, 0, {T}, 0)
result += [kernels(), tune]
""")
    assert run.count("k_integrate_mfma_ticks") < T
    assert tuned.count("k_integrate_tile") == tuned.count("k_integrate_mfma") == 2 * T
    assert "k_integrate_mfma_ticks" not in tuned
    assert tune["candidates"] == 2


def test_router_of_a_handle_without_the_byte_ring(dry):
    """In a workspace that holds everything but the byte ring, the router that the
    launch shape names is the one that runs: eight lanes per word for a few
    blocks (the automatic choice), one lane per word when asked for."""
    auto, one, tuned = dry("""
net = W.random_net(63, 8, 256, 256, 4, grid_w=4)
S, T = 3, 2
h = load(net, S, T, "plain", need(net, S, T, "plain") - (4 + 2) * S * 8 * 256)
shape = R.ranc_get_launch_shape(h)
result = [[shape["route_lanes_per_word"], kernels(run(h, T))]]
R.ranc_set_launch_shape(h, dict(shape, route_lanes_per_word=1))
result.append([R.ranc_get_launch_shape(h)["route_lanes_per_word"], kernels(run(h, T))])
tune = R.ranc_autotune(h, 0, 0, T, 0)
result.append([tune["candidates"], kernels()])
""")
    ends = ["k_fold_counts", "k_advance_tick"]
    assert auto == [8, ["k_integrate_plain", "k_route_split"] * 2 + ends]
    assert one == [1, ["k_integrate_plain", "k_route"] * 2 + ends]
    # (each candidate twice, and one of them is the eight-lane form)
    assert tuned[1].count("k_route_split") == 2 * 2
    assert tuned[1].count("k_route") == (tuned[0] - 1) * 2 * 2


def test_scheduled_spikes_move_when_the_form_changes(dry):
    """Calls through the router on a handle with the byte ring: the scheduled
    spikes move once, to the bit ring, and once back; in a batch too. Once a
    caller's graph holds a run, they are back in the byte ring after every call."""
    plain, batch, recorded = dry("""
GRAPH = R.RANC_RUN_GRAPH
net, other = W.random_net(1, 64, 128, 128, 4, grid_w=8), W.random_net(2, 3, 64, 64, 2, grid_w=3)
moves = lambda *a: [r[2] for r in run(*a) if r[0] == "launch"].count("k_move_ring")
def shape(h, lanes):
    R.ranc_set_launch_shape(h, dict(R.ranc_get_launch_shape(h), route_lanes_per_word=lanes))
h = load(net, 20, 4, "plain")
plain = [moves(h, 4)]
shape(h, 1)
plain += [moves(h, 4), moves(h, 4, GRAPH), moves(h, 1), moves(h, 4, GRAPH)]
shape(h, 8)
plain += [moves(h, 4), moves(h, 4, GRAPH)]
o = load(other, 2, 4, "plain")
batch = [moves([h, o], 4), moves([h, o], 4, GRAPH)]
shape(h, 1)
shape(o, 1)
batch += [moves([h, o], 4), moves([h, o], 4, GRAPH), moves(o, 4), moves([h, o], 4), moves(h, 4)]
shape(h, 8)
batch += [moves([h, o], 4, GRAPH), moves(h, 4)]
dry.dry_capturing(1)
recorded = [moves(h, 4, 0, 7)]
dry.dry_capturing(0)
shape(h, 1)
recorded += [moves(h, 4, 0, 7), moves(h, 4, GRAPH, 7)]
shape(h, 8)
recorded += [moves(h, 4, 0, 7)]
result = [plain, batch, recorded]
""")
    assert plain == [0, 1, 0, 0, 0, 1, 0]
    # (h has launches of its own in the batch and keeps its router there; o,
    # among the batch's kernels, is on the byte ring there and on the bit ring alone)
    assert batch == [0, 0, 1, 0, 1, 1, 0, 1, 0]
    assert recorded == [0, 2, 2, 0]


@pytest.mark.parametrize("kernel", ["k_plain_whole", "k_integrate_tile"])
def test_error_in_a_branch_of_a_batch(dry, kernel):
    """A launch that fails in one of a batch's branches: the call's error tells
    which launch and why, and every branch joins the caller's stream."""
    message, rows = dry(f"""
a, b = W.random_net(1, 4, 64, 64, 2, grid_w=2), W.random_net(2, 3, 64, 64, 2, grid_w=3)
hs = [load(a, 3, 16, "plain"), load(b, 3, 16, "plain"), load(b, 64, 16, "mfma")]
dry.dry_fail({kernel!r}.encode())
try:
    run(hs, 16)
    result = None
except R.RancError as e:
    result = [str(e), log()]
""")
    assert "out of memory" in message and ("several ticks" if kernel == "k_plain_whole" else "branches") in message
    branches = {r[1] for r in rows if r[0] == "wait" and r[1] != 0}
    joins = {r[1] for r in rows if r[0] == "record" and r[1] != 0 and ["wait", 0, r[2]] in rows}
    assert len(branches) == 3 and joins == branches


@pytest.mark.parametrize("path", ["plain", "mfma"])
def test_profile_of_a_batch_counts_every_launch(dry, path):
    """The first handle's profile holds the launches of all networks of a batch, of
    those with launches of their own too (a large plain network; a feed-forward
    one), and theirs hold none."""
    first, other, queued = dry(f"""
big = W.random_net(1, 64, 128, 128, 4, grid_w=8) if {path!r} == "plain" else forward_net(17, 4, 256, 256, 4, 9, 2)
hs = [load(W.random_net(2, 3, 64, 64, 2, grid_w=3), 2, 8, "plain"), load(big, 64 if {path!r} == "mfma" else 20, 8, {path!r})]
R.ranc_profile_enable(hs[0], True)
rows = run(hs, 8)
result = [R.ranc_profile_read(h)["integrate_launches"] for h in hs] + [kernels(rows)]
""")
    integrations = [k for k in queued if k.startswith(("k_plain_ticks", "k_integrate"))]
    assert first == len(integrations) > 8 and other == 0


def test_profile_of_many_calls_keeps_few_events(dry):
    """Profiling left on over many calls of several ticks per launch: the event
    pairs are folded into the totals from time to time and reused."""
    calls, events = dry("""
h = load(W.random_net(1, 4, 64, 64, 2, grid_w=2), 1, 16, "plain")
R.ranc_profile_enable(h, True)
rows = [r for i in range(9000) for r in run(h, 16)]
result = [R.ranc_profile_read(h)["integrate_launches"], len({r[2] for r in rows if r[0] == "record"})]
""")
    assert calls == 9000 and events <= 2 * 4097


# (cores, axons, neurons, bits, samples, types, feed-forward, path): the faster one as
# timed, on both sides of each line of the rule below 64 samples
BELOW_A_TILE = [(200, 128, 128, 9, 42, 4, False, "mfma"), (128, 256, 256, 9, 32, 4, False, "mfma"), (127, 256, 256, 9, 32, 4, False, "plain"),
                (128, 64, 256, 9, 32, 4, False, "plain"), (205, 64, 256, 9, 32, 4, False, "mfma"), (128, 64, 256, 8, 32, 4, False, "mfma"),
                (61, 128, 512, 9, 40, 4, False, "plain"), (103, 128, 512, 9, 32, 4, False, "mfma"), (64, 128, 512, 8, 32, 4, False, "mfma"),
                (64, 64, 512, 8, 32, 4, False, "plain"), (103, 64, 512, 8, 32, 4, False, "mfma"),
                (64, 64, 512, 9, 32, 4, False, "plain"), (98, 64, 512, 9, 63, 8, False, "mfma"), (124, 64, 512, 9, 63, 8, False, "mfma"),
                (192, 64, 512, 9, 32, 4, False, "plain"), (256, 64, 512, 9, 32, 8, False, "plain"), (220, 64, 512, 9, 56, 4, False, "mfma"),
                (373, 64, 512, 9, 44, 8, False, "mfma"), (373, 64, 512, 9, 44, 4, False, "plain"),
                (72, 256, 256, 9, 56, 4, True, "plain"), (116, 256, 256, 9, 56, 4, True, "mfma"), (164, 256, 256, 9, 32, 4, True, "mfma"),
                (64, 512, 512, 8, 32, 4, True, "plain"), (64, 512, 512, 8, 32, 2, True, "mfma"), (84, 512, 512, 8, 32, 4, True, "mfma"),
                (128, 512, 512, 9, 63, 4, True, "mfma"), (256, 512, 512, 9, 32, 4, True, "plain"), (184, 512, 512, 9, 44, 4, True, "plain"),
                (220, 512, 256, 9, 56, 4, True, "mfma"), (256, 512, 256, 9, 32, 4, True, "plain"),
                (64, 512, 512, 9, 48, 4, False, "mfma"), (336, 512, 128, 9, 48, 4, True, "mfma")]


def test_automatic_path_below_a_tile(dry):
    got = dry(f"""
def net(C, A, N, bits, G, forward):
    n = W.random_net(1, C, A, N, G, weight_bits=bits, grid_w=C, density=0.0, p_core=0.0 if forward else 0.5, config_id=873)
    return n
result = []
for C, A, N, bits, S, G, forward, _ in {BELOW_A_TILE!r}:
    h = load(net(C, A, N, bits, G, forward), S, 16, "auto")
    result.append({{1: "plain", 2: "mfma"}}[R.ranc_get_path(h)])
    R.ranc_free(h)
    held.clear()
""")
    assert got == [c[-1] for c in BELOW_A_TILE]


# (path, axons, neurons, bits, levels, cores per level, samples, ticks, whether
# several ticks per launch are the faster form as timed, by 20% or more)
FORMS = [("mfma", 512, 64, 8, 2, 200, 1000, 2, False), ("mfma", 512, 64, 8, 2, 200, 200, 4, False),
         ("mfma", 256, 64, 9, 2, 200, 1000, 2, False), ("mfma", 512, 128, 8, 2, 200, 200, 2, False),
         ("mfma", 64, 256, 9, 3, 64, 300, 4, True), ("mfma", 128, 128, 9, 3, 64, 300, 4, True),
         ("mfma", 256, 256, 9, 3, 64, 300, 4, True), ("mfma", 512, 128, 8, 2, 16, 1000, 4, True),
         ("mfma", 512, 128, 8, 6, 64, 64, 16, True), ("mfma", 256, 256, 9, 4, 128, 100, 32, True),
         ("plain", 64, 256, 9, 2, 200, 40, 2, False), ("plain", 256, 256, 9, 2, 200, 40, 4, True),
         ("plain", 512, 512, 9, 4, 32, 1, 32, True)]


def test_ticks_per_launch_of_feed_forward_networks(dry):
    got = dry(f"""
from tests.test_gpu_form_coverage import layers_net
result = []
for path, A, N, bits, levels, per, S, T, _ in {FORMS!r}:
    h = load(layers_net(1, levels, per, A, N, 4, bits), S, T, path)
    rows = run(h, T)
    # (all of a launch's cores: tick by tick)
    grids = {{int(r[3]) for r in rows if r[0] == "launch" and r[2] == "k_plain_ticks"}}
    result.append("k_integrate_mfma_ticks" in kernels(rows) if path == "mfma" else grids != {{levels * per}})
    R.ranc_free(h)
    held.clear()
""")
    assert got == [f[-1] for f in FORMS]


@pytest.mark.parametrize("path,S", [("plain", 20), ("mfma", 64)])
def test_reset_clears_what_can_hold_spikes(dry, path, S):
    """A reset of a feed-forward network clears the scheduler slots (or history) of
    the next max_delay ticks, not the slots that blocks of ticks need beside them;
    all of them after loading, after a call that failed and when recorded."""
    loaded, reset, failed, recorded, again = dry(f"""
net = forward_net(17, 30, 64, 256, 4, 9, 6)
d = R.Desc(net)
n = R.ranc_workspace_bytes(d, {S}, 32, R.PATHS[{path!r}])
ws = np.zeros(n + 256, np.uint8)
h = R.ranc_load_network(d, {S}, 32, R.PATHS[{path!r}], -(-ws.ctypes.data // 256) * 256, n, 0)
def cleared(rows):
    return [sum(int(r[5]) for r in rows if r[2] == "k_fill_u32"), [r[2] for r in rows].count("k_clear_slots")]
def reset(stream=0):
    R.ranc_reset_state(h, stream)
    return cleared(log())
result = [cleared(log()), reset()]
dry.dry_fail(b"k_")
try:
    run(h, 3)
except R.RancError:
    pass
dry.dry_fail(b"")
log()
result.append(reset())
dry.dry_capturing(1)
result.append(reset(7))
dry.dry_capturing(0)
result.append(reset())
""")
    C, A, N, D = 30, 64, 256, 4
    if path == "plain":
        ring = (D + 1 + 32) * S * C * A
        assert loaded[0] - reset[0] == ring // 4 + ring // 32   # (bytes, and one bit each)
        assert [x[1] for x in (loaded, reset, failed, recorded, again)] == [0, 1, 0, 0, 1]
    else:
        assert loaded[0] - reset[0] == 32 * C * N * (S // 64) * 2
    assert failed == recorded == loaded and again == reset
