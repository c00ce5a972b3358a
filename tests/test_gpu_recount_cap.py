"""The cap on the sweep-wide recount's workgroups, set once, before the first sweeps
(workgroups striding over the work, and no cap), and the cap in force set once more
between sweeps: the oracle's trajectory in both precision forms."""
import numpy as np
import pytest

from oracle import sweep as osw
import synthgen

from cases import EDGE, gpu_problem, oracle_problem, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("cap", [3, 7, 0])
def test_a_cap_before_the_first_sweep(cap, precision):
    w = dict(EDGE["n256_r4"], precision=precision)
    say("case cap", cap, precision)
    inp = synthgen.problem_inputs(w)
    ref = oracle_problem(w, inp)
    st = osw.run(ref, osw.initial_state(ref, inp["offsets"]), 7)
    with gpu_problem(w, inp) as p:
        p.set_recount_blocks(cap)
        p.sweep(2)
        p.set_recount_blocks(cap)   # the one in force: nothing changes
        p.sweep(5)
        np.testing.assert_array_equal(p.get_offsets(), st.u)
        np.testing.assert_array_equal(p.get_counts().reshape(st.c.shape), st.c)
