"""GPU parity of the cable solve at the edges of its units (backward Euler of
the cable equation, the "Other" phase of a step) against the oracle, at the
bars of tests/parity.py."""
import numpy as np
import pytest

from paper_1905_02241_amd import mech, workloads as W
from tests.parity import compare_nodes, compare_states, run_gpu, run_oracle

pytestmark = pytest.mark.gpu


def chain(n):
    p = np.arange(-1, n - 1)
    return p


def star(n):
    p = np.zeros(n, dtype=np.int64)
    p[0] = -1
    return p


def comb(stems, length):
    """A root with `stems` unbranched children of `length` nodes."""
    p = [-1]
    for _ in range(stems):
        for j in range(length):
            p.append(0 if j == 0 else len(p) - 1)
    return np.array(p)


FORESTS = {
    # rows per unit around one and two waves, a single node, an even and an odd last row
    "small": ([chain(1), chain(2), star(3), star(4), chain(63), star(64), chain(65), comb(9, 3), star(129)], 0),
    # each of them a unit of its own, cut at an odd bound
    "small-cut": ([chain(63), star(64), chain(65), comb(9, 3), star(129)], 5),
    # the largest cell that stays whole, and one node more
    "whole": ([chain(2416)], 0),
    "cut": ([chain(2417)], 0),
    # a trunk that fits LDS but not beside a piece: a launch of its own
    "trunk": ([comb(1500, 3)], 2400),
    # a trunk solved by its pieces, with more ghosts than a wave
    "ghosts": ([comb(300, 7)], 64),
}


@pytest.mark.parametrize("name", sorted(FORESTS))
def test_units_at_their_edges(name):
    trees, unit = FORESTS[name]
    parent, first = [], 0
    for t in trees:
        parent.append(np.where(t >= 0, t + first, -1))
        first += t.shape[0]
    parent = np.concatenate(parent).astype(np.int32)
    w = W.make_tiny(81, kinds=("pas", "hh"), n_nodes=first, vmode="cable", nsteps=25, shuffle=False)
    rng = np.random.default_rng(81)
    w.parent = parent
    w.g_axial = np.where(parent >= 0, rng.uniform(0.05, 0.3, first), 0.0)
    w.v_init = -60.0
    got, m = run_gpu(w, 25, "batched", "fp64", unit_nodes=unit)
    M = run_oracle(w, 25)
    compare_states(got, M, "fp64", label=name)
    compare_nodes(got, M, "fp64", label=name)
    plan = mech.cable_plan(w.parent, unit)
    cut = plan["list_top"].shape[0] + plan["list_top_g"].shape[0]
    assert cut == {"small": 0, "small-cut": 5, "whole": 0, "cut": 1, "trunk": 1, "ghosts": 1}[name]
