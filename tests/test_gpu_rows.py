"""Counts and error rows that cross to the host in more than one round of the
staging buffer (128 MiB): every row against the other call's, and sampled rows
about the rounds' boundaries against the oracle."""
import numpy as np
import pytest

from oracle import estimator
import synthgen

from cases import gpu_problem, say, workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("t,tg", [(1061, 0), (1040, 3)])
def test_rows_in_several_rounds(t, tg):
    w = workload(n=4, g=(1, 3), width=256, height=256, t_heaviside=t, t_gauss=tg, radius=1)
    say("case rows", t, tg)
    inp = synthgen.problem_inputs(w)
    with gpu_problem(w, inp) as p:
        c, e = p.get_counts(), p.get_errors()
        _, area = p.get_integrands()
    P, most = 256 * 256, 128 << 20
    assert c.nbytes > most and e.nbytes > most
    edge = {0, P - 1}
    for row in (2 * t, 4 * (t + tg)):
        per = most // row
        edge |= {r + d for r in range(per, P, per) for d in (-1, 0, 1)}
    px = np.array(sorted(edge))
    want = estimator.hit_counts(w["n"], w["g"], inp["offsets"].reshape(-1, 2)[px], inp["heaviside"])
    np.testing.assert_array_equal(c[px], want)
    # the count over N is exact: one rounding of the area, one of the difference
    exact = c / 4.0 - area
    assert np.all(np.abs(e[:, :t] - exact) <= 2.0 ** -24 * (1 + 2.0 ** -23) * (area + np.abs(exact)))
    assert np.all(np.isfinite(e))
