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
# two, both sides of the tile size's thresholds (512, 2048 and 7000 instances
# per CU of 256), and a ragged mix of types
@pytest.mark.parametrize("make,n", [("hh", 1), ("hh", 2), ("hh", 131071), ("hh", 131072), ("hh", 524287),
                                    ("hh", 524288), ("hh", 1791999), ("hh", 1792000), ("mixed", 1), ("mixed", 4097), ("mixed", 39500)])
def test_own_shape_gives_the_same_bits(make, n):
    w = W.make_c1(n_nodes=n) if make == "hh" else W.make_c5(n_nodes=n)
    steps = 5
    a, _ = run_gpu(w, steps, "batched", "fp64")
    b, _ = run_gpu(w, steps, "batched", "fp64", launch=(128, 256, 128, 0, 0))
    same(a, b)


@pytest.mark.parametrize("vmode", ["clamp", "isolated"])
@pytest.mark.parametrize("shared_ca", [0, 1])
@pytest.mark.parametrize("steps", [1, 2, 3, 256, 257, 260])
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


@pytest.mark.parametrize("model", ["hh", "mixed"])
def test_own_shape_by_name_is_the_own_shape(model):
    """What mech_get_launch reports can be set and changes nothing: a small
    context's steps stay together in one launch."""
    from paper_1905_02241_amd import mech
    w = W.make_c1(n_nodes=3000) if model == "hh" else W.make_c5(n_nodes=3000)
    shape = mech.from_workload(w, "fp64").get_launch()
    a, _ = run_gpu(w, 9, "batched", "fp64")
    b, mb = run_gpu(w, 9, "batched", "fp64", launch=shape)
    same(a, b)
    assert tuple(mb.get_launch()) == tuple(shape)


def crowded():
    """One node with more instances than a tile's LDS holds, its neighbours
    with none or a few."""
    w = W.make_tiny(83, kinds=("pas", "hh", "syn"), n_nodes=300, vmode="external", syn_per_node=2.0)
    s = w.slots[0]
    node = np.concatenate([s.node, np.full(5000, 7, dtype=np.int32)]).astype(np.int32)
    s.params["g"] = np.concatenate([s.params["g"], np.full(5000, 1e-5)])
    s.params["e"] = np.concatenate([s.params["e"], np.full(5000, -70.0)])
    w.slots[0] = W.Slot("pas", node, s.params)
    return w


PHASES = {
    "all": lambda: W.make_tiny(84, kinds=W.KINDS, n_nodes=333, per_node=2, syn_per_node=7.0, vmode="external",
                               density_fraction=0.7),
    # runs of one node longer than a wave
    "runs": lambda: W.make_tiny(85, kinds=("pas", "syn"), n_nodes=11, per_node=1, syn_per_node=150.0, vmode="external"),
    "one": lambda: W.make_tiny(86, kinds=("hh",), n_nodes=1, vmode="external"),
    "crowded": crowded,
}


@pytest.mark.parametrize("shared_ca", [0, 1])
@pytest.mark.parametrize("name", sorted(PHASES))
def test_single_phases_match_the_oracle(name, shared_ca):
    from oracle import oracle as O
    from paper_1905_02241_amd import mech
    from tests.parity import compare_nodes, compare_states
    w = PHASES[name]()
    if shared_ca and not any(s.kind in mech.CA_KINDS for s in w.slots):
        pytest.skip("no calcium type")
    w.globals["shared_ca"] = shared_ca
    m = mech.from_workload(w, "fp64")
    M = O.Model(w)
    M.init()
    rng = np.random.default_rng(9)
    for k in range(6):
        snap = {"states": mech.states_of(m), "v": m.nodes()["v"], "k": k}
        if shared_ca:
            snap["cai"] = m.ion("cai")
        m.cur(k, w.dt)
        M.events(k)
        M.cur()
        got = {**m.nodes(), "states": mech.states_of(m)}
        compare_nodes({**got, "snap": snap}, M, "fp64", label=f"{name} cur k={k}", check_v=False)
        v = rng.uniform(-80, 30, w.n_nodes)
        m.set_node_array("v", v)
        M.v[:] = v
        m.state(w.dt)
        M.state()
        compare_states({"states": mech.states_of(m)}, M, "fp64", label=f"{name} state k={k}")
    # accumulate: twice the currents of types without events
    a = m.nodes()
    if not any(s.kind == "syn" for s in w.slots):
        m.cur(7, w.dt)
        a = m.nodes()
        m.cur(7, w.dt, accumulate=True)
        b = m.nodes()
        for key in ("rhs", "d"):
            assert np.array_equal(b[key], 2.0 * a[key]), key


@pytest.mark.parametrize("shape", [(64, 64, 64, 0, 1), (256, 256, 128, 0, 1), (256, 4096, 2048, 0, 1)])
def test_single_phases_after_a_chosen_shape(shape):
    """The caller's tile table may be longer than the one it replaces: the
    single phases, which keep their own, give the bits they gave before."""
    from paper_1905_02241_amd import mech
    w = W.make_tiny(88, kinds=W.KINDS, n_nodes=3001, vmode="external", syn_per_node=2.0)

    def phases(shapes):
        m = mech.from_workload(w, "fp64")
        for k, s in enumerate(shapes):
            if s:
                m.set_launch(*s)
            m.cur(k, w.dt)
            m.state(w.dt)
        return {**m.nodes(), "states": mech.states_of(m)}
    same(phases([None] * 4), phases([None, shape, (128, 256, 64, 0, 1), shape]))


def test_resident_tile_without_room_for_the_table_of_runs():
    """A tile that fills the LDS of a workgroup to within the 2 KiB that the
    table would take: its waves find their runs by the ends."""
    n = 8150
    w = W.make_tiny(87, kinds=("pas",), n_nodes=1, vmode="isolated")
    rng = np.random.default_rng(87)
    w.slots[0] = W.Slot("pas", np.zeros(n, dtype=np.int32),
                        {"g": rng.uniform(1e-7, 2e-7, n), "e": rng.uniform(-80.0, -60.0, n)})
    shape = (1024, 16384, 64, 0, 1)
    a, _ = run_gpu(w, 20, "batched", "fp64", launch=shape)
    b, _ = run_gpu(w, 20, "resident", "fp64", launch=shape, resident_steps=6)
    same(a, b)
