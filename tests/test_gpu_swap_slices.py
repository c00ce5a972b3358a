"""Swap passes whose integrands go in several slices: one stage a slice, several of
several, a short last one, and counts on uint16 rows whose sums bound the stages of
a slice; trajectories equal the oracle's."""
import dataclasses

import numpy as np
import pytest

from oracle import sweep as osw
import synthgen

from cases import gpu_problem, oracle_problem, say, workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,g,t,side,r", [(16, (1, 7), 100, 8, 2), (16, (1, 7), 1030, 16, 3), (16, (1, 7), 3000, 8, 6),
                                          (1024, (1, 1023), 700, 8, 1), (4096, (1, 1365), 900, 8, 2)])
def test_sliced_passes_match_the_oracle(n, g, t, side, r):
    w = workload(n=n, g=g, t_heaviside=t, width=side, height=side, radius=r, move=1)
    say("case swap slices", n, t, side)
    inp = synthgen.problem_inputs(w)
    ref = dataclasses.replace(oracle_problem(w, inp), move=1)
    st = osw.initial_state(ref, inp["offsets"])
    with gpu_problem(w, inp) as p:
        p.phase_evaluate(0)
        got, want = p.get_swap_pass(), osw.swap_pass(ref, osw.initial_state(ref, inp["offsets"]), 0)
        np.testing.assert_array_equal(got["delta"], want["delta"])
        p.sweep(3)
        osw.run(ref, st, 3)
        np.testing.assert_array_equal(p.get_offsets(), st.u)
        np.testing.assert_array_equal(p.get_counts(), st.c.reshape(-1, t))
