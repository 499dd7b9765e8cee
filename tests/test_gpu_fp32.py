"""FP32-mixed on the launch structures that the library chooses by itself: the
single phases against the oracle at the FP32 bars of tests/parity.py, and
several steps a launch against a launch per step, bit for bit (every instance
is updated by the same code, and node sums in fixed point do not depend on the
order of the adds)."""
import dataclasses

import numpy as np
import pytest

from paper_1905_02241_amd import workloads as W
from tests.parity import compare_nodes, compare_states, run_gpu
from tests.test_gpu_launch import PHASES, same

pytestmark = pytest.mark.gpu


def as_stored(w):
    """The workload with the PARAMETERs that FP32-mixed keeps in float rounded
    to it: near v = e a rounded reversal potential (up to 5e-6 mV off) is more
    of g (v - e) than the current update's own rounding."""
    slots = [W.Slot(s.kind, s.node, {k: a if s.kind == "syn" else a.astype(np.float32).astype(np.float64)
                                     for k, a in s.params.items()}) for s in w.slots]
    return dataclasses.replace(w, slots=slots)


@pytest.mark.parametrize("name,shared_ca", [(n, 0) for n in sorted(PHASES)] + [("all", 1)])
def test_single_phases_match_the_oracle(name, shared_ca):
    from oracle import oracle as O
    from paper_1905_02241_amd import mech
    w = PHASES[name]()
    w.globals["shared_ca"] = shared_ca
    m = mech.from_workload(w, "fp32")
    M = O.Model(as_stored(w))
    M.init()
    rng = np.random.default_rng(10)
    for k in range(6):
        snap = {"states": mech.states_of(m), "v": m.nodes()["v"], "k": k}
        if shared_ca:
            snap["cai"] = m.ion("cai")
        m.cur(k, w.dt)
        M.events(k)
        M.cur()
        got = {**m.nodes(), "states": mech.states_of(m)}
        compare_nodes({**got, "snap": snap}, M, "fp32", label=f"{name} cur k={k}", check_v=False)
        v = rng.uniform(-80, 30, w.n_nodes)
        m.set_node_array("v", v)
        M.v[:] = v
        m.state(w.dt)
        M.state()
        compare_states({"states": mech.states_of(m)}, M, "fp32", label=f"{name} state k={k}")


@pytest.mark.parametrize("vmode", ["clamp", "isolated"])
@pytest.mark.parametrize("shared_ca", [0, 1])
@pytest.mark.parametrize("steps", [1, 3, 257])
def test_several_steps_a_launch_give_the_same_bits(vmode, shared_ca, steps):
    w = W.make_tiny(82, kinds=W.KINDS, n_nodes=777, vmode=vmode, syn_per_node=5.0, event_rate_hz=300.0)
    w.globals["shared_ca"] = shared_ca
    a, ma = run_gpu(w, steps, "batched", "fp32")
    b, mb = run_gpu(w, steps, "batched", "fp32", launch=(128, 256, 128, 0, 0))
    same(a, b)
    for name in ("cai", "ica"):
        assert np.array_equal(ma.ion(name), mb.ion(name)), name


@pytest.mark.parametrize("n", [4097, 39500])
def test_own_shape_gives_the_same_bits(n):
    """Types that the smaller kernels take (no buffered calcium, no node ion)."""
    w = W.make_c5(n_nodes=n)
    a, _ = run_gpu(w, 40, "batched", "fp32")
    b, _ = run_gpu(w, 40, "batched", "fp32", launch=(128, 256, 128, 0, 0))
    same(a, b)
