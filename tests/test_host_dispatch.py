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
