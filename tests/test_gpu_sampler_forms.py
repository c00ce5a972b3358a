"""Sampler queries at the edges of the kernel's blocks and of the staging
buffer: queries about multiples of a workgroup's, pairs about a run of eight and
a launch's 32, results larger than the buffer, an output on an odd float; and
reads of the same problem's rows between queries."""
import ctypes as C

import numpy as np
import pytest
import torch

from oracle import estimator, sampler
import synthgen

from cases import say

pytestmark = pytest.mark.gpu
bnlat = pytest.importorskip("paper_2105_12620_amd.bnlat")


def pairs_of(count):
    probs, pairs = [], []
    for mw in synthgen.dimension_pair_batch(count=count, seed=9, t=8, radius=1):
        mw = dict(mw, width=16, height=12)
        inp = dict(synthgen.problem_inputs(mw))
        p = bnlat.create_problem(mw, bnlat.heaviside_array(inp["heaviside"]))
        p.init_offsets(inp["offsets"])
        probs.append(p)
        pairs.append(dict(n=mw["n"], g=mw["g"], width=16, height=12, u=inp["offsets"]))
    return probs, pairs


def queries(m):
    g = np.random.default_rng(m)
    return [g.integers(0, hi, m).astype(np.uint32) for hi in (5000, 5000, 1 << 20)]


@pytest.mark.parametrize("count,m", [(1, 1), (7, 255), (8, 256), (9, 257), (32, 300), (33, 513), (20, 430000)])
def test_queries_equal_the_oracles(count, m):
    say("case sample", count, m)
    probs, pairs = pairs_of(count)
    x, y, k = queries(m)
    some = np.unique(np.concatenate([np.arange(min(m, 600)), np.arange(max(0, m - 300), m)]))
    want = sampler.sample_q16(pairs, x[some], y[some], k[some]) / 65536.0
    for _ in range(2):   # the second finds the buffer there
        np.testing.assert_array_equal(bnlat.sample(probs, x, y, k)[some].astype(np.float64), want)
        probs[0].compute_errors()
        c = probs[0].get_counts()   # the same buffer
        u = pairs[0]["u"].reshape(-1, 2).astype(np.int64)
        h = {f: probs[0].get_integrands()[0][f] for f in ("nx", "ny", "cx", "cy")}
        np.testing.assert_array_equal(c, estimator.hit_counts(pairs[0]["n"], pairs[0]["g"], u, h))
    for p in probs:
        p.close()


def test_device_query_into_an_odd_float():
    probs, pairs = pairs_of(3)
    x, y, k = queries(777)
    dev = [torch.as_tensor(a.astype(np.int32)).cuda() for a in (x, y, k)]
    out = torch.full((777 * 6 + 3,), -1.0, device="cuda")
    torch.cuda.synchronize()
    arr = (C.c_void_p * 3)(*[p.handle.value for p in probs])
    bnlat._call("bn_sample_device", arr, 3, *[C.c_void_p(d.data_ptr()) for d in dev], 777,
                C.c_void_p(out.data_ptr() + 4), None)
    got = out.cpu().numpy()
    np.testing.assert_array_equal(got[1:-2].reshape(777, 6).astype(np.float64),
                                  sampler.sample_q16(pairs, x, y, k) / 65536.0)
    assert got[0] == got[-1] == got[-2] == -1.0
    for p in probs:
        p.close()
