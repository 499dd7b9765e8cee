"""The single current update (BREAKPOINT, section 3 of the paper) where a node
carries many instances of a type: node sums against the oracle, and their cost."""
import numpy as np
import pytest

from paper_1905_02241_amd import workloads as W
from tests.parity import compare_nodes

pytestmark = pytest.mark.gpu


def with_synapses(counts, seed=91, kinds=("pas", "cahva")):
    """Synapses in the given numbers on nodes 0, 1, ... of a small mesh."""
    w = W.make_tiny(seed, kinds=kinds, n_nodes=200, vmode="external", event_rate_hz=20000.0)
    rng = np.random.default_rng(seed)
    node = np.repeat(np.arange(len(counts)), counts).astype(np.int32)
    w.slots.append(W.Slot("syn", node, {"weight": rng.uniform(0.1, 2.0, node.shape[0])}))
    return w


def crowded_channels():
    """Calcium channels past a wave on one node: the node's calcium current too."""
    w = W.make_tiny(92, kinds=("pas", "cahva"), n_nodes=60, vmode="external")
    s = w.slots[1]
    w.slots[1] = W.Slot("cahva", np.concatenate([s.node, np.full(200, 5)]).astype(np.int32),
                        {"gbar": np.concatenate([s.params["gbar"], np.linspace(1e-6, 5e-6, 200)])})
    return w


# both sides of one and two waves and of the length that a wave sums, a run that ends a tile, one that fills it,
# and nodes without any between them
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("case", ["edges", "gaps", "tile", "calcium"])
def test_long_runs_match_the_oracle(case, prec):
    from oracle import oracle as O
    from paper_1905_02241_amd import mech
    w = {"edges": lambda: with_synapses([63, 64, 65, 79, 80, 81, 127, 128, 129, 1, 300]),
         "gaps": lambda: with_synapses([0, 80, 0, 0, 700, 2, 0, 80]),
         "tile": lambda: with_synapses([2500, 1, 1100, 1024]),
         "calcium": crowded_channels}[case]()
    w.globals["shared_ca"] = 1 if case == "calcium" else 0
    m = mech.from_workload(w, prec)
    M = O.Model(w)
    M.init()
    v = np.random.default_rng(5).uniform(-20, 30, w.n_nodes)   # away from every reversal potential
    m.set_node_array("v", v)
    M.v[:] = v
    for k in range(3):
        snap = {"states": mech.states_of(m), "v": v, "k": k}
        if case == "calcium":
            snap["cai"] = m.ion("cai")
        m.cur(k, w.dt)
        got = {**m.nodes(), "states": mech.states_of(m)}
        compare_nodes({**got, "snap": snap}, M, prec, label=f"{case} k={k}", check_v=False)
        first = m.nodes()
    if case == "calcium":
        M.cur()
        # FP32: 2e-3 of the magnitudes (the bar of the node's calcium current)
        assert np.allclose(m.ion("ica"), M.ica_node, rtol=1e-11 if prec == "fp64" else 2e-3, atol=0)
        m.cur(3, w.dt)
        assert np.array_equal(m.nodes()["rhs"], first["rhs"])   # the same bits on every run


def test_a_crowded_node_costs_what_spread_instances_cost():
    """2000 synapses on one node against the same number over 200 nodes.  A
    thread that sums them one after the other takes 200 us more than either
    launch; both launches are below 20."""
    import torch
    from paper_1905_02241_amd import mech

    def us(counts):
        m = mech.from_workload(with_synapses(counts), "fp64")
        for k in range(10):
            m.cur(k, 0.025)
        times = []
        for _ in range(7):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record(m.stream)
            for k in range(50):
                m.cur(k, 0.025)
            b.record(m.stream)
            b.synchronize()
            times.append(a.elapsed_time(b) * 20.0)
        return sorted(times)[3]
    assert us([2000]) < 3.0 * us([10] * 200)
