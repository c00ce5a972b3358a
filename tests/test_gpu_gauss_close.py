"""Which estimates decide a move on a tile with line estimates: within the margin
those sample by sample of its whole window, as they are on a tile too small for
the line form, else the lines'.  Gaussians so wide that g is near 1, hence read
back exactly from the FP32 error vectors (g - I is small): of the tile (lines), of
a tile of the proposals (lines) and of small tiles of each tested move's window
(samples).  The energy change is the Heaviside part, exact, and the Gaussian part
from the FP32 estimates of one form or the other, in FP64 (up to 2^-47 of the sum
of its terms' sizes); the two differ by many times that."""
import numpy as np
import pytest

import synthgen

from cases import gpu_problem, say, workload

pytestmark = pytest.mark.gpu
bnlat = pytest.importorskip("paper_2105_12620_amd.bnlat")

W, H, R = 48, 46, 2


def values(p, t):
    """FP32 estimates behind a problem's error vectors, exactly."""
    integrals = p.get_integrands(gaussians=True)[3]
    e = p.get_errors()[:, t:].astype(np.float64)
    g = (e + integrals).astype(np.float32).astype(np.float64)
    assert np.all(np.abs(e) < g / 4)
    return g


@pytest.mark.parametrize("n,g,t", [(16, (1, 7), 1), (256, (1, 79), 2), (2048, (1, 717), 1)])
def test_close_moves_take_the_samples_estimates(n, g, t):
    tg = 130
    w = workload(n=n, g=g, width=W, height=H, t_heaviside=t, t_gauss=tg, radius=R)
    inp = synthgen.problem_inputs(w)
    inp["gauss"]["s"][:] = np.linspace(8.0, 120.0, tg)
    if n == 2048:   # counts of 2048 samples nearly always change: an edge that none of them meets
        for k, v in dict(nx=11585, ny=11585, cx=0, cy=0).items():
            inp["heaviside"][k][:] = v
    say("case close", n)
    kappa = 3
    with gpu_problem(w, inp) as p:
        tile = values(p, t).reshape(H, W, tg)
        c0 = p.get_counts().reshape(H, W, t).astype(np.float64)
        p.phase_propose(kappa)
        p.phase_evaluate(kappa)
        ph = p.get_phase()
        d2, wc = bnlat.window_classes(p.cfg)
        moved = inp["offsets"].reshape(H, W, 2).copy()
        moved[1::2, 1::2] = ph["u_new"].reshape(H // 2, W // 2, 2)
        p.init_offsets(moved)
        p.compute_errors()
        new = values(p, t).reshape(H, W, tg)
    weight = dict(zip(d2.tolist(), wc.tolist()))
    off = [(oy, ox) for oy in range(-R, R + 1) for ox in range(-R, R + 1) if oy or ox]
    wd = np.array([weight[oy * oy + ox * ox] for oy, ox in off])

    def part(gm, go, gn):
        d, x = gn - go, gn + go - 2 * gm
        terms = 2 * wd[:, None] * d * x
        return np.sum(terms.astype(np.longdouble)), np.sum(np.abs(terms)), d, x

    js = synthgen.pixel_sample((W // 2) * (H // 2), 48, 5).tolist()
    u = inp["offsets"].reshape(H, W, 2)
    small = workload(n=n, g=g, width=len(off) + 2, height=len(js), t_heaviside=t, t_gauss=tg, radius=1, colour_k=1)
    seen = {"close": 0, "far": 0, "told apart": 0}
    samples = []
    for at in range(0, len(js), 4):   # tiles of four windows stay below the line form
        group = js[at:at + 4]
        rows = []
        for j in group:
            y, x = 1 + 2 * (j // (W // 2)), 1 + 2 * (j % (W // 2))
            rows.append([u[(y + oy) % H, (x + ox) % W] for oy, ox in off] + [u[y, x], ph["u_new"][j]])
        sw = dict(small, height=len(group))
        si = dict(inp, offsets=np.array(rows, dtype=np.uint16))
        with gpu_problem(sw, si) as q:
            samples += list(values(q, t).reshape(len(group), len(off) + 2, tg))
    for j, s in zip(js, samples):
        y, x = 1 + 2 * (j // (W // 2)), 1 + 2 * (j % (W // 2))
        cm = np.array([c0[(y + oy) % H, (x + ox) % W] for oy, ox in off])
        cn, co = ph["c_new"][j].astype(np.float64), c0[y, x]
        hv = np.longdouble(2) * np.sum(wd[:, None].astype(np.longdouble) * (cn - co) * (cn + co - 2 * cm)) / (n * n)
        gm = np.array([tile[(y + oy) % H, (x + ox) % W] for oy, ox in off])
        line, size, d, xm = part(gm, tile[y, x], new[y, x])
        samp, size2, _, _ = part(s[:-2], s[-2], s[-1])
        W_, b, sm = wd.sum(), (wd[:, None] * xm * xm).sum(axis=0), tile[y, x] + new[y, x]
        r, ad = np.sqrt(W_ * b), np.abs(d)
        margin = np.sum(2 * 2.0 ** -24 * 1.01 * ((W_ * ad + r) * (1.48 + 22 * sm) + 11 * (b + ad * r)))
        total = hv + line
        tol = 2.0 ** -47 * (size + size2) + 2.0 ** -51 * abs(hv)
        got = np.longdouble(ph["delta"][j])
        if abs(total) <= 0.98 * margin:
            assert abs(got - (hv + samp)) <= tol, (j, float(got - hv - samp), float(tol))
            seen["close"] += 1
            seen["told apart"] += abs(samp - line) > 8 * tol
        elif abs(total) >= 1.02 * margin:
            assert abs(got - total) <= tol, (j, float(got - total), float(tol))
            seen["far"] += 1
        assert ph["accept"][j] == (ph["delta"][j] < 0)
    say(n, seen)
    assert seen["close"] >= 3 and seen["told apart"] >= 2 and (seen["far"] >= 3 or n == 2048)
