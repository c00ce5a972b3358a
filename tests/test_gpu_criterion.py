"""Blur criterion, spectrum and energy at the edges of their kernels' blocks:
tiles whose sides are no multiple of 16 outputs or 8 frequencies (or shorter),
runs of taps shorter and longer than a block, one and several chunks of
integrands, few and many shares of the energy's tiles."""
import numpy as np
import pytest

from oracle import quality, sweep as osw
import synthgen

from cases import gpu_problem, oracle_problem, say, workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("w,h,t,r", [(4, 4, 5, 1), (16, 16, 64, 3), (20, 36, 65, 2), (12, 8, 600, 6), (48, 24, 130, 4)])
def test_criteria_equal_the_oracles(w, h, t, r):
    wl = workload(n=16, g=(1, 7), width=w, height=h, t_heaviside=t, radius=r, colour_k=1)
    say("case criterion", w, h, t, r)
    inp = synthgen.problem_inputs(wl)
    ref = oracle_problem(wl, inp)
    st = osw.initial_state(ref, inp["offsets"])
    e = osw.errors(ref, st)
    sig = [0.25, 0.7, 1.5, 4.0, 20.0]
    nbins = max(w, h)
    with gpu_problem(wl, inp) as p:
        q, en, (power, bins) = p.quality_metric(sig), p.energy(), p.error_spectrum(nbins)
    eps = 2.0 ** -24
    top = np.abs(e).max()
    # taps sum to 1 and each pass adds at most n of them (roundings of the taps,
    # the errors and the sums): |b - exact| <= (w + h + 6) eps max|e|
    want = quality.quality(e, sig)
    assert np.all(np.abs(q - want) <= (w + h + 6) * eps * top)
    assert en == pytest.approx(osw.energy_of(ref, st), rel=1e-12)
    pw, cnt = quality.error_spectrum(e, nbins)
    np.testing.assert_array_equal(bins, cnt)
    # a frequency's value is off by at most (2 (w + h) + 8) eps sum |e_t|
    err = (2 * (w + h) + 8) * eps * np.abs(e).sum(axis=(0, 1)).max()
    amp = np.sqrt(pw * w * h)
    assert np.all(np.abs(power - pw) <= (2 * amp * err + err * err) / (w * h) + 1e-30)
