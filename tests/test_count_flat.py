"""The line counter's flat edges (nearly along the lattice lines, and short normals)
against the direct count of the samples, on the library's own tables: every N it
serves, good and degenerate generators, normals of every length, edges through
samples; every product n . b1 from 0 on either side up to the limit is met."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def model(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("flat") / "libflat.so")
    subprocess.run(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-ffp-contract=off",
                    os.path.join(HERE, "count_flat_model.cpp"), "-o", out], check=True)
    return C.CDLL(out)


def rows(n, g, k, rng):
    step = 65536 // n
    nx, ny = np.zeros(k, np.int64), np.zeros(k, np.int64)
    q = k // 3
    # short normals
    nx[:q], ny[:q] = rng.integers(-6, 7, q), rng.integers(-6, 7, q)
    # across short lattice vectors, scaled, off by up to two
    s = rng.integers(1, n + 1, k - q)
    vx, vy = (s * g[0] + n // 2) % n - n // 2, (s * g[1] + n // 2) % n - n // 2
    size = np.maximum(1, np.maximum(abs(vx), abs(vy)))
    keep = size < max(2.0, 2.5 * n ** 0.5)
    f = np.where(keep, rng.integers(1, 16001, k - q) // size, 1)
    nx[q:] = np.clip(-vy * f + rng.integers(-2, 3, k - q), -16384, 16384)
    ny[q:] = np.clip(vx * f + rng.integers(-2, 3, k - q), -16384, 16384)
    zero = (nx == 0) & (ny == 0)
    nx[zero] = 1
    c = rng.integers(0, 65536, (2, k), dtype=np.uint16)
    u = rng.integers(0, 65536, (2, k), dtype=np.uint16)
    u[:, ::5] = rng.choice([0, 1, step - 1, 65535], (2, len(u[0, ::5])))
    i = rng.integers(0, n, k)
    on = rng.random(k) < 0.5
    c[0][on] = (u[0] + i * g[0] % n * step)[on].astype(np.uint16)
    c[1][on] = (u[1] + i * g[1] % n * step)[on].astype(np.uint16)
    return nx.astype(np.int16), ny.astype(np.int16), c[0].copy(), c[1].copy(), u[0].copy(), u[1].copy()


@pytest.mark.parametrize("n", [16, 64, 256, 512, 1024, 2048, 4096])
def test_flat_counts_equal_direct_counts(model, n):
    rng = np.random.default_rng(n)
    gens = [(1, 1), (1, n - 1), (1, 3), (1, n // 2 + 1), (1, int(n * 0.618) | 1), (1, int(n * 0.37) | 1)]
    k, flat = 3000 if n <= 1024 else 800, 0
    for g in gens:
        a = rows(n, g, k, rng)
        got, want = np.zeros(k, np.uint32), np.zeros(k, np.uint32)
        few = model.count_flat_model(n, g[0], g[1], k, *[x.ctypes.data_as(C.c_void_p) for x in a],
                                     got.ctypes.data_as(C.c_void_p), want.ctypes.data_as(C.c_void_p))
        assert few >= 0
        np.testing.assert_array_equal(got, want, err_msg=f"g={g}")
        flat += few
    assert flat > 50
