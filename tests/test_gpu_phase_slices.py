"""Colour phases whose integrands are split over workgroups: integrand counts on
both sides of the first that is split, ones that leave the last slice short or its
last stage ragged, many slices of few stages and few of many, in every operand form
(int8 narrow and split, uint16, the BF16 forms with and without Gaussian rows) and
colour modulus, alone and in a batch whose members need different numbers of
slices; trajectories equal the oracle's."""
import numpy as np
import pytest

from oracle import sweep as osw
import synthgen

from cases import gpu_problem, oracle_problem, say, workload

pytestmark = pytest.mark.gpu
bnlat = pytest.importorskip("paper_2105_12620_amd.bnlat")

CASES = {
    "below": dict(t_heaviside=704),
    "first": dict(t_heaviside=705),
    "ragged": dict(t_heaviside=1000, radius=1, objective=-1),
    "odd_stages": dict(t_heaviside=64 * 13, radius=6),
    "k1": dict(t_heaviside=770, colour_k=1, width=12, height=20),
    "k4": dict(t_heaviside=1025, colour_k=4, radius=4),
    "many": dict(t_heaviside=4500, width=8, height=8, radius=2),
    "few_of_many": dict(t_heaviside=780, n=1, g=(1, 1), width=160, height=152, radius=1),
    "split": dict(t_heaviside=900, n=128, g=(1, 1)),
    "wide": dict(t_heaviside=900, n=512, g=(1, 1), width=12, height=12),
    "wide_k1_r5": dict(t_heaviside=773, n=512, g=(1, 1), width=12, height=12, colour_k=1, radius=5),
    "bf16": dict(t_heaviside=900, precision=1),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_split_phases_match_the_oracle(name):
    w = workload(**CASES[name])
    say("case slices", name)
    inp = synthgen.problem_inputs(w)
    ref = oracle_problem(w, inp)
    st = osw.initial_state(ref, inp["offsets"])
    with gpu_problem(w, inp) as p:
        for kappa in range(w["colour_k"] ** 2):
            p.phase_propose(kappa)
            p.phase_evaluate(kappa)
            got, want = p.get_phase(), osw.phase(ref, st, kappa)
            np.testing.assert_array_equal(got["delta"], want["delta"])
            np.testing.assert_array_equal(got["accept"], want["accept"])
            p.phase_commit(kappa)
        p.phase_advance()
        st.sweep += 1
        p.sweep(3)
        osw.run(ref, st, 3)
        np.testing.assert_array_equal(p.get_offsets(), st.u)
        np.testing.assert_array_equal(p.get_counts(), st.c.reshape(-1, w["t_heaviside"]))


@pytest.mark.parametrize("tg", [0, 64])
def test_split_approximate_bf16_takes_exact_moves(tg):
    """What the approximate BF16 form takes, re-evaluated on split integrands, has
    the exact energy change (Heaviside rows: equal; a Gaussian's FP32 estimates are
    within 2^-20 of the exact ones, its part within 8 of those for each unit of
    window weight)."""
    w = workload(n=512, g=(1, 189), t_heaviside=770, t_gauss=tg, width=12, height=12, precision=1)
    say("case slices bf16", tg)
    inp = synthgen.problem_inputs(w)
    ref = oracle_problem(w, inp)
    with gpu_problem(w, inp) as p:
        p.phase_propose(0)
        p.phase_evaluate(0)
        got = p.get_phase()
    want = osw.phase(ref, osw.initial_state(ref, inp["offsets"]), 0)
    took = got["accept"]
    assert took.any()
    weight = sum(np.exp(-(x * x + y * y) / w["sigma"] ** 2) for x in range(-3, 4) for y in range(-3, 4) if x or y)
    np.testing.assert_allclose(got["delta"][took], want["delta"][took], rtol=1e-12, atol=tg * 8 * weight * 2.0 ** -20)


def test_members_of_a_batch_have_their_own_slices():
    kinds = [dict(t_heaviside=705), dict(t_heaviside=40), dict(t_heaviside=2100, width=8, height=8),
             dict(t_heaviside=1500, n=512, g=(1, 1)), dict(t_heaviside=800, n=128, g=(1, 1), radius=2)]
    ws = [workload(problem_id=i, **k) for i, k in enumerate(kinds)]
    torch = pytest.importorskip("torch")
    stream = torch.cuda.Stream()
    ps, refs, sts = [], [], []
    for w in ws:
        inp = synthgen.problem_inputs(w)
        p = bnlat.create_problem(w, bnlat.heaviside_array(inp["heaviside"]), stream=stream.cuda_stream)
        p.init_offsets(inp["offsets"])
        p.compute_errors()
        ps.append(p)
        refs.append(oracle_problem(w, inp))
        sts.append(osw.initial_state(refs[-1], inp["offsets"]))
    say("case slices batch")
    with bnlat.Batch(ps) as b:
        b.sweep(3)
        for p, w, ref, st in zip(ps, ws, refs, sts):
            osw.run(ref, st, 3)
            np.testing.assert_array_equal(p.get_offsets(), st.u)
            np.testing.assert_array_equal(p.get_counts(), st.c.reshape(-1, w["t_heaviside"]))
    for p in ps:
        p.close()
