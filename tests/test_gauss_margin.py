"""The margin within which moves on line estimates are decided again (gauss_margin in
csrc/kernels.hip), on the CPU: the sample by sample form's estimate (FP64 exponents
rounded to FP32, FP32 exponentials, eight FP32 additions at a time), emulated with
NumPy's FP32 exp2 and the exponential's documented error of one unit in the last
place on top, is within 2^-24 (0.37 + 10 g) of the exact one, and moves' parts from
the two forms differ by less than the margin."""
import numpy as np
import pytest

from oracle import estimator
import synthgen


def sample_form(n, g, u, table, worse):
    """The estimates [P, T]; worse: sign of a unit in the last place on every term."""
    x = estimator.shifted_points(n, g, u).astype(np.float64) / 65536.0   # [P, N, 2]
    out = np.empty((u.shape[0], len(table["s"])))
    # index i of the lattice: lane i % 64 adds i, i + 64, ... in groups of eight
    chunk = 512
    for k, (mx, my, s) in enumerate(zip(table["mx"], table["my"], table["s"])):
        a = np.log2(np.e) / (2 * s * s)
        e = -a * (x[..., 0] ** 2 + x[..., 1] ** 2) + 2 * a * (mx * x[..., 0] + my * x[..., 1]) - a * (mx * mx + my * my)
        f = np.exp2(e.astype(np.float32))
        f = np.nextafter(f, np.float32(worse * np.inf)).astype(np.float32) if worse else f
        total = np.zeros(u.shape[0])
        for c in range(0, n, chunk):
            part = np.zeros((u.shape[0], 64), np.float32)
            for q in range(0, min(chunk, n - c), 64):
                v = f[:, c + q:c + min(q + 64, n - c)]
                part[:, :v.shape[1]] += v
            total += part.astype(np.float64).sum(axis=1)
        out[:, k] = (total / n).astype(np.float32)
    return out


@pytest.mark.parametrize("n,g", [(16, (1, 7)), (256, (1, 79)), (1024, (1, 381))])
@pytest.mark.parametrize("worse", [-1, 0, 1])
def test_margin_covers_both_forms(n, g, worse):
    rng = np.random.default_rng(n + worse)
    table = {k: v.copy() for k, v in synthgen.gaussian_table(24, 4).items()}
    table["s"][::4] = [0.5, 1.0, 3.0, 10.0, 40.0, 0.02]
    R, sigma = 2, 2.1
    off = [(y, x) for y in range(-R, R + 1) for x in range(-R, R + 1) if x or y]
    w = np.exp(-np.array([y * y + x * x for y, x in off]) / sigma ** 2)
    for _ in range(6):
        u = rng.integers(0, 65536, (len(off) + 2, 2))
        exact = estimator.gauss_estimates(n, g, u, table)
        samp = sample_form(n, g, u, table, worse)
        assert np.all(np.abs(samp - exact) <= 2.0 ** -24 * (0.37 + 10 * exact))
        line = exact.astype(np.float32).astype(np.float64)

        def part(e):
            d, x = e[-1] - e[-2], e[-1] + e[-2] - 2 * e[:-2]
            return 2 * np.sum(w[:, None] * d * x, axis=0), np.abs(d), np.sum(w[:, None] * x * x, axis=0), e[-1] + e[-2]

        pl, d, b, s = part(line)
        ps = part(samp)[0]
        W = w.sum()
        r = np.sqrt(W * b) * (1 + 1e-12)
        margin = 2.0 * 2.0 ** -24 * 1.01 * ((W * d + r) * (1.48 + 22.0 * s) + 11.0 * (b + d * r))
        # the two forms' second-order difference (products of estimates' errors) is
        # below 4 W (4 eta(1))^2
        assert np.all(np.abs(pl - ps) <= margin + 64 * W * (2.0 ** -24 * 11.37) ** 2)
