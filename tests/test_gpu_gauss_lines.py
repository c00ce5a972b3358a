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


@pytest.mark.parametrize("n,g", [(16, (1, 7)), (256, (1, 79)), (1024, (1, 381)), (4096, (1, 1365))])
def test_close_moves_are_decided_again(n, g):
    """Gaussians so wide that their part of the energy change is of the size of
    its rounding: moves that leave the one Heaviside's count as it is are within
    the line form's margin and decided from estimates sample by sample.  Energy
    changes stay within that margin of the exact ones, and each decision is its
    energy change's sign."""
    w = workload(n=n, g=g, width=48, height=46, t_heaviside=1, t_gauss=130, radius=2)
    inp = synthgen.problem_inputs(w)
    inp["gauss"]["s"][:] = np.linspace(40.0, 400.0, 130)
    say("close", n)
    with gpu_problem(w, inp) as p:
        p.phase_propose(3)
        p.phase_evaluate(3)
        ph = p.get_phase()
        c0 = p.get_counts().reshape(46, 48)
        p.phase_propose(3)   # the list of the first evaluation is spent
        p.phase_evaluate(3)
        again = p.get_phase()
    for k in ("delta", "accept"):
        np.testing.assert_array_equal(ph[k], again[k])
    np.testing.assert_array_equal(ph["accept"].astype(bool), ph["delta"] < 0)
    u = inp["offsets"].reshape(46, 48, 2).astype(np.int64)
    close = 0
    for j in synthgen.pixel_sample(24 * 23, 40, 5):
        y, x = 1 + 2 * (int(j) // 24), 1 + 2 * (int(j) % 24)
        off = [(oy, ox) for oy in range(-2, 3) for ox in range(-2, 3) if oy or ox]
        q = np.array([u[(y + oy) % 46, (x + ox) % 48] for oy, ox in off] + [u[y, x], ph["u_new"].reshape(-1, 2)[j].astype(np.int64)])
        e = estimator.gauss_estimates(n, g, q, inp["gauss"])
        c = np.array([c0[(y + oy) % 46, (x + ox) % 48] for oy, ox in off] + [c0[y, x], ph["c_new"].reshape(-1)[j]]) / n
        wd = np.exp(-np.array([oy * oy + ox * ox for oy, ox in off]) / w["sigma"] ** 2)
        d, xm = e[-1] - e[-2], e[-1] + e[-2] - 2 * e[:-2]
        exact = 2 * np.sum(wd[:, None] * d * xm) + 2 * np.sum(wd * (c[-1] - c[-2]) * (c[-1] + c[-2] - 2 * c[:-2]))
        margin = 8 * 11.4 * 2.0 ** -24 * np.sum(wd[:, None] * (np.abs(xm) + np.abs(d))) * 1.1
        # the estimates' own rounding (half a unit, g <= 1) where x and d are below it
        margin += 2 * 130 * wd.sum() * (4 * 2.0 ** -24) ** 2 * 16
        assert abs(ph["delta"][j] - exact) <= margin + 1e-12 * abs(exact), (j, ph["delta"][j], exact, margin)
        close += abs(exact) <= margin
    assert close > 0 or n == 4096   # the counts of 4096 samples nearly always change
