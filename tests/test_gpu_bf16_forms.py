"""The BF16 form with exact counts on either operand: int8 where the counts'
bound allows (trajectory, per-phase values and the BF16 field's energy equal the
oracle's), BF16 where it does not (near-axis lattices, at every colour modulus)."""
import numpy as np
import pytest

from oracle import sweep as osw
import synthgen

from cases import gpu_problem, oracle_problem, say, workload

pytestmark = pytest.mark.gpu

CASES = {
    "bf16_axis_k1": workload(n=256, g=(1, 1), t_heaviside=40, width=12, height=12, colour_k=1),
    "bf16_axis_k2": workload(n=256, g=(1, 1), t_heaviside=130, width=20, height=12, radius=4),
    "bf16_axis_k4": workload(n=256, g=(1, 255), t_heaviside=17, width=16, height=16, radius=2, colour_k=4),
    "int8_narrow": workload(n=256, g=(1, 79), t_heaviside=70, width=20, height=12, radius=4),
    "int8_split": workload(n=128, g=(1, 1), t_heaviside=33, colour_k=4),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_exact_bf16_form_equals_the_oracle(name):
    w = dict(CASES[name], precision=1)
    say(name)
    inp = synthgen.problem_inputs(w)
    ref = oracle_problem(w, inp)
    st = osw.initial_state(ref, inp["offsets"])
    with gpu_problem(w, inp) as p:
        for kappa in range(w["colour_k"] ** 2):
            p.phase_propose(kappa)
            p.phase_evaluate(kappa)
            got, raw = p.get_phase(), p.get_phase_bf16()
            ph = osw.phase(ref, st, kappa)
            np.testing.assert_array_equal(got["accept"], ph["accept"])
            np.testing.assert_allclose(got["delta"], ph["delta"], rtol=1e-12, atol=0)
            # N sum |dc| < 2^24 at these sizes: the pass's own value is exact too
            np.testing.assert_allclose(raw, ph["delta"], rtol=1e-12, atol=0)
            p.phase_commit(kappa)
        p.phase_advance()
        st.sweep += 1
        stats = p.sweep(3, stats=True)
        assert stats["bf16_vetoes"] == 0
        osw.run(ref, st, 3)
        np.testing.assert_array_equal(p.get_offsets(), st.u)
        np.testing.assert_array_equal(p.get_counts(), st.c.reshape(-1, w["t_heaviside"]))
        assert p.energy_bf16() == pytest.approx(osw.energy_of(ref, st), rel=1e-12)
        p.sweep(1)
        osw.run(ref, st, 1)
        assert p.energy_bf16() == pytest.approx(osw.energy_of(ref, st), rel=1e-12)
