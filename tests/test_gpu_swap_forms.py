"""Swap passes on int8 deviations and on counts (chosen by the counts' bound)
give the oracle's trajectory at the edges of the blocks, stages and slices:
one and several stages, slices and rounds of members, few and many integrands
a word, radii with and without column steps."""
import numpy as np
import pytest

from oracle import sweep as osw
import synthgen

from cases import gpu_problem, say, workload

pytestmark = pytest.mark.gpu

CASES = {
    "int8_n1": workload(n=1, g=(1, 1), t_heaviside=17),
    "int8_n64_k1": workload(n=64, g=(1, 1), t_heaviside=40, colour_k=1),      # every pixel a member: several rounds
    "int8_n256_wide_tile": workload(n=256, g=(1, 79), t_heaviside=129, width=64, height=16, radius=4),
    "int8_n256_r6": workload(n=256, g=(1, 79), t_heaviside=300, width=16, height=16, radius=6),
    "counts_n128_axis": workload(n=128, g=(1, 1), t_heaviside=70, radius=2),
    "counts_n1024_r5": workload(n=1024, g=(1, 381), t_heaviside=260, width=32, height=16, radius=5),
    "counts_n4096_k1": workload(n=4096, g=(1, 1), t_heaviside=33, width=32, height=8, radius=1, colour_k=1),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_swap_trajectory_equals_the_oracles(name):
    w = dict(CASES[name], move=1)
    say(name)
    inp = synthgen.problem_inputs(w)
    ref = osw.Problem(n=w["n"], g=w["g"], width=w["width"], height=w["height"], radius=w["radius"], sigma=w["sigma"],
                      colour_k=w["colour_k"], seed=w["seed"], problem_id=w["problem_id"], table=inp["heaviside"],
                      objective=1, move=1)
    st = osw.initial_state(ref, inp["offsets"])
    with gpu_problem(w, inp) as p:
        for k in (2, 1):
            p.sweep(k)
            osw.run(ref, st, k)
            np.testing.assert_array_equal(p.get_offsets(), st.u)
            np.testing.assert_array_equal(p.get_counts(), st.c.reshape(-1, w["t_heaviside"]))
        p.compute_errors()   # from the offsets alone
        np.testing.assert_array_equal(p.get_counts(), st.c.reshape(-1, w["t_heaviside"]))
