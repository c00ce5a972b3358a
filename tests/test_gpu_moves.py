"""Energy changes of explicit moves at the edges of their kernel's steps: every
radius (rows and columns of steps), tiles smaller than the window, one plane
group of integrands and several, counts up to N = 4096; against the oracle's
exact value."""
import numpy as np
import pytest

from oracle import energy, estimator
import synthgen

from cases import gpu_problem, say, workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("r,w,h,n,t", [(1, 5, 6, 16, 130), (2, 4, 8, 64, 8), (3, 12, 20, 8, 300), (4, 5, 8, 256, 64),
                                       (5, 18, 14, 4096, 129), (6, 16, 14, 1024, 70)])
def test_moves_equal_the_oracles(r, w, h, n, t):
    g = {4096: (1, 1365), 1024: (1, 381), 256: (1, 79)}.get(n, (1, 3))
    wl = workload(n=n, g=g, width=w, height=h, t_heaviside=t, radius=r, colour_k=1)
    say("case moves", r, w, h, n, t)
    inp = synthgen.problem_inputs(wl)
    u = inp["offsets"].reshape(-1, 2).astype(np.int64)
    c = estimator.hit_counts(n, g, u, inp["heaviside"]).reshape(h, w, t)
    m = min(w * h, 37)
    px, new = synthgen.pixel_sample(w * h, m, 3), synthgen.proposals(m, 4)
    with gpu_problem(wl, inp) as p:
        delta, counts = p.delta_energy(px, new, counts=True)
    want = estimator.hit_counts(n, g, new.astype(np.int64), inp["heaviside"])
    np.testing.assert_array_equal(counts, want)
    d = energy.delta_exact(c, px // w, px % w, want, n, r, wl["sigma"])
    np.testing.assert_allclose(delta, d, rtol=1e-12, atol=0)
