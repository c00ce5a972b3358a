"""The line counter (hit counts from one clamped crossing per lattice line)
against the direct count of the samples, on the library's own tables: every N
it serves, generators of every kind, offsets and edges chosen so that samples
lie on or next to the edge."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

from oracle import integrands

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def model(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("lines") / "libmodel.so")
    subprocess.run(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-ffp-contract=off",
                    os.path.join(HERE, "count_lines_model.cpp"), "-o", out], check=True)
    return C.CDLL(out)


def rows(n, k, g, rng):
    theta = rng.uniform(0, 2 * np.pi, k)
    nx = np.rint(16384 * np.cos(theta)).astype(np.int16)
    ny = np.rint(16384 * np.sin(theta)).astype(np.int16)
    q = k // 4
    # axis-parallel and diagonal edges, tiny and extreme normals
    nx[:q], ny[:q] = rng.choice([-16384, -1, 0, 1, 16384], q), rng.choice([-16384, -2, 1, 3, 16384], q)
    # edges nearly along short lattice vectors
    step = 65536 // n
    s = rng.integers(1, n + 1, q)
    vx, vy = (s * g[0] + n // 2) % n - n // 2, (s * g[1] + n // 2) % n - n // 2
    f = 16000 // np.maximum(1, np.maximum(abs(vx), abs(vy)))
    nx[q:2 * q], ny[q:2 * q] = -vy * f + rng.integers(-1, 2, q), vx * f
    zero = (nx == 0) & (ny == 0)
    nx[zero] = 1
    c = rng.integers(0, 65536, (2, k), dtype=np.uint16)
    u = rng.integers(0, 65536, (2, k), dtype=np.uint16)
    # offsets on the grid's corners, and edge points on a sample of the pixel
    u[:, ::5] = rng.choice([0, 1, step - 1, 65535], (2, len(u[0, ::5])))
    i = rng.integers(0, n, k)
    on = rng.random(k) < 0.5
    c[0][on] = (u[0] + i * g[0] % n * step)[on].astype(np.uint16)
    c[1][on] = (u[1] + i * g[1] % n * step)[on].astype(np.uint16)
    return nx, ny, c[0].copy(), c[1].copy(), u[0].copy(), u[1].copy()


@pytest.mark.parametrize("n", [16, 32, 64, 128, 256, 512, 1024, 2048, 4096])
def test_line_counts_equal_direct_counts(model, n):
    rng = np.random.default_rng(n)
    gens = [(1, 1), (1, n - 1), (1, 3), (3, 1), (1, n // 2 + 1), (1, n // 2 - 1), (1, int(n * 0.618) | 1)]
    gens += [(int(2 * rng.integers(0, n // 2) + 1), int(2 * rng.integers(0, n // 2) + 1)) for _ in range(24)]
    k, by_sample = 4000 if n <= 1024 else 1000, 0
    for g in gens:
        a = rows(n, k, g, rng)
        got, want, few = np.zeros(k, np.uint32), np.zeros(k, np.uint32), C.c_uint32()
        lines = model.count_lines_model(n, g[0], g[1], k, *[x.ctypes.data_as(C.c_void_p) for x in a],
                                        got.ctypes.data_as(C.c_void_p), want.ctypes.data_as(C.c_void_p), C.byref(few))
        assert 0 < lines <= (2 * n) ** 0.5
        np.testing.assert_array_equal(got, want, err_msg=f"g={g}")
        by_sample += few.value
    assert 0 < by_sample < 0.5 * k * len(gens)


@pytest.mark.parametrize("n", [16, 64, 256, 1024, 4096])
def test_every_generator_has_lines(model, n):
    """Each lattice of N points is that of (1, y) for an odd y: its line table
    exists for all of them (every 16th at the largest N), and padded integrands
    count nothing."""
    for y in range(1, n, 2 if n <= 1024 else 32):
        assert model.count_lines_padding(n, 1, y) == 0, y


@pytest.mark.parametrize("n", [128, 256, 512, 1024, 2048])
def test_counts_stay_within_the_lines_bound(model, n):
    """|count - round(N area)| of random and nearly lattice-aligned edges stays
    within the bound, and the bound is of use for good generators."""
    rng = np.random.default_rng(n + 1)
    gens = [(1, 1), (1, int(n * 0.618) | 1)] + [(1, int(2 * rng.integers(0, n // 2) + 1)) for _ in range(6)]
    k = 2000
    for g in gens:
        bound = model.count_lines_deviation(n, g[0], g[1])
        a = rows(n, k, g, rng)
        got, want, few = np.zeros(k, np.uint32), np.zeros(k, np.uint32), C.c_uint32()
        model.count_lines_model(n, g[0], g[1], k, *[x.ctypes.data_as(C.c_void_p) for x in a],
                                got.ctypes.data_as(C.c_void_p), want.ctypes.data_as(C.c_void_p), C.byref(few))
        areas = np.array([integrands.heaviside_area(*(int(x[i]) for x in a[:4])) for i in range(k)])
        assert np.abs(want.astype(int) - np.rint(n * areas).astype(int)).max() <= bound, g
    assert model.count_lines_deviation(256, 1, 79) <= 63
    assert model.count_lines_deviation(1024, 1, 381) <= 126


@pytest.mark.parametrize("n", [16, 64, 256, 1024, 4096])
def test_gauss_line_sums_equal_direct_sums(model, n):
    """The Gaussian estimates along the lines against the sum over the samples,
    both in 64 bits: the drawn range of centres and widths, centres outside the
    square and narrow Gaussians up to where the table declines.  A term carries
    at most some hundred roundings of 2^-53 relative each (steps of a line,
    lines, four exponentials of exponents up to 1000: 2^-43 for those)."""
    rng = np.random.default_rng(n + 7)
    k = 300 if n <= 1024 else 60
    for g in [(1, 1 + 2 * (n // 8)), (1, int(n * 0.618) | 1), (3, 2 * int(rng.integers(0, n // 2)) + 1)]:
        mx, my = rng.uniform(0, 1, k), rng.uniform(0, 1, k)
        mx[::7] += rng.choice([-0.5, 0.5])
        s = rng.uniform(0.05, 0.3, k)
        s[1::5] = rng.uniform(0.01, 0.06, len(s[1::5]))
        s[2::11] = 3.0
        u = rng.integers(0, 65536, (2, k), dtype=np.uint16)
        got, want, few = np.zeros(k), np.zeros(k), C.c_uint32()
        args = (mx, my, s, u[0].copy(), u[1].copy())
        p = [x.ctypes.data_as(C.c_void_p) for x in args]
        steps = model.gauss_lines_model(n, g[0], g[1], k, *p, got.ctypes.data_as(C.c_void_p),
                                        want.ctypes.data_as(C.c_void_p), C.byref(few))
        assert 0 < steps <= n
        assert 0 < few.value < k / 3
        np.testing.assert_allclose(got, want, rtol=2.0 ** -40)
