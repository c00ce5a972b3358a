"""Error spectrum of tiles with one long side: at and around 2^16, where the
product of a position and a frequency no longer fits 32 bits, along x and along
y, and a ragged one whose twiddles come from a matrix, against the oracle's FFT.  A sequential FP32 sum of n terms of size a is off
by about 2^-25 a n (root mean square: partial sums grow as the square root of
their length, their roundings add at random), relative to the result's a
sqrt(n) by 2^-25 sqrt(n) = 8e-6, so a bin's power by under 1e-4."""
import numpy as np
import pytest

from oracle import quality, sweep as osw
import synthgen

from cases import gpu_problem, oracle_problem, say, workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("w,h,t", [(65528, 2, 3), (65536, 2, 3), (70000, 2, 3), (2, 70000, 3), (101, 60, 300)])
def test_spectrum_of_long_tiles(w, h, t):
    wl = workload(n=16, g=(1, 7), width=w, height=h, t_heaviside=t, radius=1, colour_k=1)
    say("case long spectrum", w, h)
    inp = synthgen.problem_inputs(wl)
    ref = oracle_problem(wl, inp)
    e = osw.errors(ref, osw.initial_state(ref, inp["offsets"]))
    with gpu_problem(wl, inp) as p:
        got, cnt = p.error_spectrum(min(w, h) + 1)
    want, bins = quality.error_spectrum(e, min(w, h) + 1)
    np.testing.assert_array_equal(cnt, bins)
    np.testing.assert_allclose(got, want, rtol=1e-4)
