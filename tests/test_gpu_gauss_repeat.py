"""A colour phase evaluated once more after its commit, on a tile with line
estimates: the moves that it took propose the offsets that their pixels have by
now, change nothing, exactly, and are not taken again."""
import numpy as np
import pytest

import synthgen

from cases import gpu_problem, say, workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,g,t,k", [(16, (1, 7), 20, 2), (2048, (1, 717), 8, 1)])   # int8 and uint16 operands
def test_taken_moves_change_nothing(n, g, t, k):
    w = workload(n=n, g=g, width=48, height=46, t_heaviside=t, t_gauss=130, colour_k=k)
    say("case repeat", n)
    inp = synthgen.problem_inputs(w)
    with gpu_problem(w, inp) as p:
        p.phase_propose(0)
        p.phase_evaluate(0)
        first = p.get_phase()
        p.phase_commit(0)
        p.phase_propose(0)
        p.phase_evaluate(0)
        again = p.get_phase()
    np.testing.assert_array_equal(first["u_new"], again["u_new"])
    taken = first["accept"]
    assert taken.any()
    np.testing.assert_array_equal(again["delta"][taken], 0.0)
    assert not again["accept"][taken].any()
