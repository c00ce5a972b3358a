"""Hit counts of edges nearly along the lattice's lines and of short normals, beside
ordinary ones in the same groups of eight, on tiles and pixel lists, against the
oracle's direct counts."""
import numpy as np
import pytest

from oracle import estimator
import synthgen

from cases import say, workload

pytestmark = pytest.mark.gpu
bnlat = pytest.importorskip("paper_2105_12620_amd.bnlat")


@pytest.mark.parametrize("n,g", [(16, (1, 7)), (64, (1, 1)), (256, (1, 79)), (1024, (1, 1023)), (4096, (1, 1365))])
def test_flat_edges(n, g):
    w = workload(n=n, g=g, width=10, height=8, t_heaviside=75)
    say("case flat", n)
    rng = np.random.default_rng(n)
    table = synthgen.heaviside_table(75, 3)
    few = np.flatnonzero(rng.random(75) < 0.6)
    pairs = [(1, 0), (0, -1), (1, -1), (-1, -1), (2, 1), (-3, 5), (16384, -16384), (7, 0), (g[1] % 50, -1), (5, 5)]
    for i in few:
        table["nx"][i], table["ny"][i] = pairs[rng.integers(len(pairs))]
    u = synthgen.offsets(10, 8, 5)
    with bnlat.create_problem(w, bnlat.heaviside_array(table)) as p:
        p.init_offsets(u)
        p.compute_errors()
        want = estimator.hit_counts(n, g, u.reshape(-1, 2).astype(np.int64), table)
        np.testing.assert_array_equal(p.get_counts(), want)
        new = synthgen.offsets(10, 8, 6).reshape(-1, 2)
        _, got = p.delta_energy(np.arange(80, dtype=np.uint32), new, counts=True)
        np.testing.assert_array_equal(got, estimator.hit_counts(n, g, new.astype(np.int64), table))
