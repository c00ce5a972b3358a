"""A caller that owns offsets and counts puts an earlier state of the problem back
into them, in stream order: sweeps, phase steps and batched sweeps go on from it
as the oracle does, in the forms whose phases read int8 copies of the counts
(narrow and split) and in the one that reads them themselves (uint16)."""
import numpy as np
import pytest

from oracle import sweep as osw
import synthgen

from cases import oracle_problem, say, workload

pytestmark = pytest.mark.gpu
bnlat = pytest.importorskip("paper_2105_12620_amd.bnlat")
torch = pytest.importorskip("torch")

FORMS = {
    "narrow": dict(n=16, g=(1, 7), t_heaviside=20),
    "split": dict(n=128, g=(1, 1), t_heaviside=130),
    "wide": dict(n=512, g=(1, 1), t_heaviside=20),
}


@pytest.mark.parametrize("how", ["sweep", "steps", "batch"])
@pytest.mark.parametrize("form", sorted(FORMS))
def test_sweeps_follow_a_restored_state(form, how):
    w = workload(width=16, height=16, **FORMS[form])
    say("restore", form, how)
    inp = synthgen.problem_inputs(w)
    ref = oracle_problem(w, inp)
    P, Tp = 256, (w["t_heaviside"] + 127) // 128 * 128
    u = torch.zeros(P, dtype=torch.int32, device="cuda")
    c = torch.zeros((Tp // 8, P, 8), dtype=torch.int16, device="cuda")
    stream = torch.cuda.Stream()
    torch.cuda.synchronize()
    st = osw.initial_state(ref, inp["offsets"])
    p = bnlat.create_problem(w, bnlat.heaviside_array(inp["heaviside"]), stream=stream.cuda_stream,
                             buffers=(u.data_ptr(), c.data_ptr(), None))
    p.init_offsets(inp["offsets"])
    p.compute_errors()
    b = bnlat.Batch([p]) if how == "batch" else None
    with torch.cuda.stream(stream):
        u0, c0 = u.clone(), c.clone()

    def go(k):
        if how == "batch":
            b.sweep(k)
        elif how == "sweep":
            p.sweep(k)
        else:
            for _ in range(k):
                for kappa in range(w["colour_k"] ** 2):
                    p.phase_propose(kappa)
                    p.phase_evaluate(kappa)
                    p.phase_commit(kappa)
                p.phase_advance()
        osw.run(ref, st, k)
        np.testing.assert_array_equal(p.get_offsets(), st.u)
        np.testing.assert_array_equal(p.get_counts(), st.c.reshape(P, -1))

    go(3)
    with torch.cuda.stream(stream):   # back to the start, at the present sweep
        u.copy_(u0)
        c.copy_(c0)
    at = st.sweep
    st = osw.initial_state(ref, inp["offsets"])
    st.sweep = at
    go(2)
    half = torch.arange(P, device="cuda") % 2 == 0   # half of the pixels once more
    torch.cuda.synchronize()
    cnt = st.c.reshape(P, -1)
    first = osw.initial_state(ref, inp["offsets"])
    even = np.arange(P) % 2 == 0
    st.u.reshape(P, 2)[even] = first.u.reshape(P, 2)[even]
    cnt[even] = first.c.reshape(P, -1)[even]
    with torch.cuda.stream(stream):
        u[half] = u0[half]
        c[:, half] = c0[:, half]
    go(1)
    if b:
        b.close()
    p.close()
