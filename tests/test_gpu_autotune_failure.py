"""A search for a launch shape that finds none leaves the context as it was."""
import numpy as np
import pytest

from paper_1905_02241_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [None, (128, 256, 128, 0, 0)])
def test_a_failed_search_keeps_both_paths_shapes(shape):
    """9000 instances on one node: 180 kB of LDS on the time-fused path at any
    shape.  The batched path's shape and tiles are the same before and after,
    and so are its results."""
    from paper_1905_02241_amd import mech
    w = W.make_tiny(93, kinds=("pas",), n_nodes=3000, vmode="isolated")
    s = w.slots[0]
    rng = np.random.default_rng(93)
    w.slots[0] = W.Slot("pas", np.concatenate([s.node, np.full(9000, 7)]).astype(np.int32),
                        {"g": np.concatenate([s.params["g"], rng.uniform(1e-7, 2e-7, 9000)]),
                         "e": np.concatenate([s.params["e"], rng.uniform(-80.0, -60.0, 9000)])})

    def run(search):
        m = mech.from_workload(w, "fp64")
        if shape:
            m.set_launch(*shape)
        before = (m.get_launch(), m.info())
        if search:
            with pytest.raises(mech.MechError):
                m.autotune(w.dt, w.vmode, 2, 1, path="resident")
        assert (m.get_launch(), m.info()) == before
        m.step(5, 0, w.dt, w.vmode, "batched")
        m.cur(5, w.dt)
        return m.nodes()
    a, b = run(False), run(True)
    for key in a:
        assert np.array_equal(a[key], b[key]), key
