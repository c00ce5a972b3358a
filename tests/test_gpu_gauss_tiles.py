"""Gaussian part of the energy change in tiles of 8 x 8 (or 8 x 4) class pixels:
launches of enough blocks to take them, ragged in both directions, at the
smallest and largest window of every colour modulus, with padded Gaussians;
sampled pixels (all corners among them) against FP64 sums over the oracle's
estimates.  A FP32 estimate is within eta = 2^-24 11.4 of the exact one, so a
Gaussian's part is within 8 eta sum_m w_m (|x_m| + |d|)."""
import numpy as np
import pytest

from oracle import estimator
import synthgen

from cases import gpu_problem, say, workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("w,h,k,r", [(130, 126, 1, 1), (128, 130, 1, 6), (260, 252, 2, 1), (260, 252, 2, 5),
                                     (256, 260, 2, 6), (368, 360, 4, 1), (364, 368, 4, 5), (368, 360, 4, 6)])
def test_gaussian_parts_equal_the_oracles(w, h, k, r):
    wl = workload(n=4, g=(1, 3), width=w, height=h, t_heaviside=1, t_gauss=70, radius=r, colour_k=k)
    say("case gauss tiles", w, h, k, r)
    inp = synthgen.problem_inputs(wl)
    kappa = k * k - 1
    with gpu_problem(wl, inp) as p:
        c0 = p.get_counts().reshape(h, w)
        p.phase_propose(kappa)
        p.phase_evaluate(kappa)
        ph = p.get_phase()
    u = inp["offsets"].reshape(h, w, 2).astype(np.int64)
    cw, ch = w // k, h // k
    js = [0, cw - 1, (ch - 1) * cw, ch * cw - 1] + [int(j) for j in synthgen.pixel_sample(cw * ch, 20, 6)]
    off = [(oy, ox) for oy in range(-r, r + 1) for ox in range(-r, r + 1) if oy or ox]
    wd = np.exp(-np.array([oy * oy + ox * ox for oy, ox in off]) / wl["sigma"] ** 2)
    for j in js:
        y, x = kappa // k + k * (j // cw), kappa % k + k * (j % cw)
        q = np.array([u[(y + oy) % h, (x + ox) % w] for oy, ox in off] + [u[y, x], ph["u_new"].reshape(-1, 2)[j].astype(np.int64)])
        e = estimator.gauss_estimates(4, (1, 3), q, inp["gauss"])
        c = np.array([c0[(y + oy) % h, (x + ox) % w] for oy, ox in off] + [c0[y, x], ph["c_new"].reshape(-1)[j]]) / 4
        d, xm = e[-1] - e[-2], e[-1] + e[-2] - 2 * e[:-2]
        exact = 2 * np.sum(wd[:, None] * d * xm) + 2 * np.sum(wd * (c[-1] - c[-2]) * (c[-1] + c[-2] - 2 * c[:-2]))
        tol = 8 * 11.4 * 2.0 ** -24 * 1.01 * np.sum(wd[:, None] * (np.abs(xm) + np.abs(d))) + 1e-12 * (1 + abs(exact))
        assert abs(ph["delta"][j] - exact) <= tol, (j, ph["delta"][j], exact, tol)
