"""The recount index follows the sweep counter through every order of calls that
move it: even and odd sweep counts, phase steps, a set counter (back, ahead and
to where it was), a batch's sweeps and a new start."""
import numpy as np
import pytest

from oracle import sweep as osw
import synthgen

from cases import gpu_problem, oracle_problem, say, workload

pytestmark = pytest.mark.gpu
bnlat = pytest.importorskip("paper_2105_12620_amd.bnlat")


def test_trajectory_through_every_way_to_move_the_counter():
    w = workload(n=16, g=(1, 7), width=16, height=12, t_heaviside=20)
    inp = synthgen.problem_inputs(w)
    ref = oracle_problem(w, inp)
    st = osw.initial_state(ref, inp["offsets"])

    def check(p):
        np.testing.assert_array_equal(p.get_offsets(), st.u)
        np.testing.assert_array_equal(p.get_counts(), st.c.reshape(-1, w["t_heaviside"]))
        assert p.get_sweep_index() == st.sweep

    def sweep(p, k):
        say("sweep", k)
        p.sweep(k)
        osw.run(ref, st, k)
        check(p)

    def steps(p):
        for kappa in range(w["colour_k"] ** 2):
            p.phase_propose(kappa)
            p.phase_evaluate(kappa)
            p.phase_commit(kappa)
        p.phase_advance()
        osw.run(ref, st, 1)
        check(p)

    def jump(p, to):
        p.set_sweep_index(to)
        st.sweep = to

    with gpu_problem(w, inp) as p:
        for k in (2, 4, 1, 2, 3, 2, 2):
            sweep(p, k)
        steps(p)
        sweep(p, 2)
        at = st.sweep
        for to in (at + 5, 3, at, at - 1, at):
            jump(p, to)
            sweep(p, 2)
        jump(p, st.sweep)
        sweep(p, 4)
        b = bnlat.Batch([p])
        for k in (2, 1):
            b.sweep(k)
            osw.run(ref, st, k)
            check(p)
        b.close()
        sweep(p, 2)
        p.init_offsets(inp["offsets"])
        p.compute_errors()
        fresh = osw.initial_state(ref, inp["offsets"])
        fresh.sweep, st = st.sweep, fresh
        sweep(p, 2)
        sweep(p, 2)
