"""The launch shapes and launch structures that the library chooses by itself:
they change no bit of the FP64 results (the node sums are order-independent,
every instance is updated by the same code)."""
import numpy as np
import pytest

from paper_1905_02241_amd import workloads as W
from tests.parity import run_gpu

pytestmark = pytest.mark.gpu


def same(a, b):
    for key in ("v", "rhs", "d"):
        assert np.array_equal(a[key], b[key]), key
    for sa, sb in zip(a["states"], b["states"]):
        for name in sa:
            assert np.array_equal(sa[name], sb[name]), name
    if "spikes" in a and a["spikes"] is not None:
        assert np.array_equal(a["spikes"], b["spikes"])


# instances: a context of one node (no room for a second tile table) and of
# two, both sides of the tile size's thresholds (512, 2048 and 5000 instances
# per CU of 256), and a ragged mix of types
@pytest.mark.parametrize("make,n", [("hh", 1), ("hh", 2), ("hh", 131071), ("hh", 131072), ("hh", 524287),
                                    ("hh", 524288), ("hh", 1280001), ("mixed", 1), ("mixed", 4097), ("mixed", 39500)])
def test_own_shape_gives_the_same_bits(make, n):
    w = W.make_c1(n_nodes=n) if make == "hh" else W.make_c5(n_nodes=n)
    steps = 5
    a, _ = run_gpu(w, steps, "batched", "fp64")
    b, _ = run_gpu(w, steps, "batched", "fp64", launch=(128, 256, 128, 0, 0))
    same(a, b)


@pytest.mark.parametrize("vmode", ["clamp", "isolated"])
@pytest.mark.parametrize("shared_ca", [0, 1])
@pytest.mark.parametrize("steps", [2, 3, 260])
def test_several_steps_a_launch_give_the_same_bits(vmode, shared_ca, steps):
    """Every type, ragged tiles, from no middle step to more than one launch
    holds, against a launch per step (a shape set by the caller)."""
    w = W.make_tiny(82, kinds=W.KINDS, n_nodes=777, vmode=vmode, syn_per_node=5.0, event_rate_hz=300.0)
    w.globals["shared_ca"] = shared_ca
    a, ma = run_gpu(w, steps, "batched", "fp64")
    b, mb = run_gpu(w, steps, "batched", "fp64", launch=(128, 256, 128, 0, 0))
    same(a, b)
    for name in ("cai", "ica"):
        assert np.array_equal(ma.ion(name), mb.ion(name)), name
