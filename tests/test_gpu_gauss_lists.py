"""Energy changes of listed moves on tiles whose Gaussian estimates come from
lattice lines, in lists on both sides of the length from which theirs do too: a
move to the offset that its pixel has changes nothing, exactly; a move's change
in a short list is that in the whole one but for the two forms' rounding; and the
allocation-free entry point gives the same.

An estimate g is off by at most eta(g) = 2^-24 (0.37 + 11 g) from one form to the
other, so the Gaussian part 2 sum w (g' - g)(g' + g - 2 g_m) by at most
2 sum w (|x_m| + |d|) eta(1) <= 2 W 3 eta(1) for each of the Gaussians (W the sum of
the weights, |x_m| <= 2, |d| <= 1)."""
import numpy as np
import pytest

import synthgen

from cases import gpu_problem, say, workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,g,tg", [(16, (1, 7), 260), (256, (1, 79), 250), (1024, (1, 381), 256)])
def test_listed_moves(n, g, tg):
    w = workload(n=n, g=g, width=48, height=46, t_heaviside=8, t_gauss=tg)
    say("case gauss lists", n)
    inp = synthgen.problem_inputs(w)
    P = 48 * 46
    rng = np.random.default_rng(n)
    px = rng.permutation(P).astype(np.uint32)
    new = rng.integers(0, 65536, (P, 2), dtype=np.uint16)
    own = inp["offsets"].reshape(-1, 2)[px]
    W = sum(np.exp(-(x * x + y * y) / w["sigma"] ** 2) for x in range(-3, 4) for y in range(-3, 4) if x or y)
    tol = tg * 6 * W * 2.0 ** -24 * 11.37
    with gpu_problem(w, inp) as p:
        every = p.delta_energy(px, new)
        np.testing.assert_array_equal(p.delta_energy(px, own), np.zeros(P))
        for m in (1, 5, 64, 65, 300):
            short = p.delta_energy(px[:m], new[:m])
            np.testing.assert_array_equal(p.delta_energy_noalloc(px[:m], new[:m]), short)
            np.testing.assert_allclose(short, every[:m], rtol=0, atol=tol)
            np.testing.assert_array_equal(p.delta_energy(px[:m], own[:m]), np.zeros(m))
