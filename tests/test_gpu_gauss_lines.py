"""Gaussian estimates along lattice lines: tiles large enough to take that form,
with N at both ends of its range, padded Gaussians, pixels past a whole wave, a
lattice whose lines are too long for it, and Gaussians whose exponents leave its
range, against the oracle's FP64 sums (an estimate is rounded once to FP32: half
a unit in the last place, 2^-24 relative)."""
import numpy as np
import pytest

from oracle import estimator
import synthgen

from cases import gpu_problem, say, workload

pytestmark = pytest.mark.gpu

CASES = {
    "n16": workload(n=16, g=(1, 7), width=48, height=44, t_heaviside=8, t_gauss=130),
    "n16_diagonal": workload(n=16, g=(1, 1), width=48, height=48, t_heaviside=8, t_gauss=120),
    "n256_ragged": workload(n=256, g=(3, 79), width=50, height=46, t_heaviside=8, t_gauss=120),
    "n1024": workload(n=1024, g=(1, 381), width=48, height=46, t_heaviside=8, t_gauss=128),
    "n1024_long_lines": workload(n=1024, g=(1, 1), width=48, height=46, t_heaviside=8, t_gauss=128),
    "n4096": workload(n=4096, g=(1, 1365), width=46, height=46, t_heaviside=8, t_gauss=128),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_estimates_equal_the_oracles(name):
    w = CASES[name]
    inp = synthgen.problem_inputs(w)
    g = inp["gauss"]
    g["s"][::9] = [0.012, 0.03, 0.05, 2.0][len(name) % 4]   # narrow ones leave the form's range
    g["mx"][3] = 1.4
    say(name)
    with gpu_problem(w, inp) as p:
        got = p.get_errors()[:, w["t_heaviside"]:].astype(np.float64)
        integrals = p.get_integrands(gaussians=True)[3]
    pix = synthgen.pixel_sample(got.shape[0], 400 if w["n"] <= 256 else 60, 3)
    u = inp["offsets"].reshape(-1, 2).astype(np.int64)[pix]
    want = estimator.gauss_estimates(w["n"], w["g"], u, g)
    # the error vector g - I rounds once more; terms under 2^-126 count as 0
    # where they are summed in FP32
    tol = 2.0 ** -24 * (np.maximum(want, 2.0 ** -126) + np.abs(want - integrals)) * 1.01
    by_sample = name == "n1024_long_lines" or g["s"].min() < 0.04
    if by_sample:   # FP32 exponentials of 2^-23 relative, each
        tol = tol + 2.0 ** -22 * want
    assert np.all(np.abs(got[pix] - (want - integrals)) <= tol + 2.0 ** -126)
