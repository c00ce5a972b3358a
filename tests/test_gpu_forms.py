"""The operands of the colour phases (uint16 counts, int8 deviations, int8
deviations with changes beyond int8): trajectories equal the oracle's at the
sizes where each is chosen and at its edges: few and many integrands a word,
one and several slices, tiles smaller than a block, every colour modulus."""
import numpy as np
import pytest

from oracle import sweep as osw
import synthgen

from cases import gpu_problem, oracle_problem, say, workload

pytestmark = pytest.mark.gpu

CASES = {
    "narrow_n1": workload(n=1, g=(1, 1), t_heaviside=17),
    "narrow_n8_ragged": workload(n=8, g=(1, 3), t_heaviside=129, radius=2, colour_k=1),
    "narrow_n64_axis": workload(n=64, g=(1, 1), t_heaviside=40),
    "narrow_n256_k4": workload(n=256, g=(1, 79), t_heaviside=48, width=16, height=24, radius=4, colour_k=4),
    "narrow_n256_r6": workload(n=256, g=(1, 79), t_heaviside=16, width=14, height=14, radius=6),
    "split_n128_axis": workload(n=128, g=(1, 1), t_heaviside=70),
    "split_n1024": workload(n=1024, g=(1, 381), t_heaviside=33, width=12, height=12, radius=5),
    "split_n1024_k1": workload(n=1024, g=(1, 381), t_heaviside=20, width=8, height=8, colour_k=1),
    "wide_n256_axis": workload(n=256, g=(1, 1), t_heaviside=40, width=12, height=12),
    "wide_n4096": workload(n=4096, g=(1, 1), t_heaviside=9, width=8, height=8, radius=2),
    "modulus_3": workload(n=64, g=(1, 19), t_heaviside=40, width=12, height=12, colour_k=3),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_trajectory_equals_the_oracles(name):
    w = CASES[name]
    inp = synthgen.problem_inputs(w)
    say(name)
    p = gpu_problem(w, inp)
    ref = oracle_problem(w, inp)
    st = osw.initial_state(ref, inp["offsets"])
    for k in (3, 2):   # an odd count, then a replayed pair
        p.sweep(k)
        osw.run(ref, st, k)
        np.testing.assert_array_equal(p.get_offsets(), st.u)
        np.testing.assert_array_equal(p.get_counts(), st.c.reshape(-1, w["t_heaviside"]))
        assert p.get_sweep_index() == st.sweep
    p.close()
