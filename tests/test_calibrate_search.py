"""The calibration's search for delta, run on the host with the code that the GPU runs: how many rounds it takes, and what it finds."""
import ctypes

import numpy as np
import pytest

import oracle as O
import paper_2603_24840_amd as A


def f32(x):
    return float(np.float32(x))


def search(c_pos, c_neg, args):
    c_pos, c_neg = np.ascontiguousarray(c_pos, np.int64), np.ascontiguousarray(c_neg, np.int64)
    rounds, delta = ctypes.c_int32(), ctypes.c_double()
    assert A.lib().arrol_calibrate_search(c_pos.ctypes.data, c_neg.ctypes.data, len(c_pos), A.Policy(*args), ctypes.byref(rounds), ctypes.byref(delta)) == 0
    return rounds.value, delta.value


# A round is a sum over the bins, one behind the other: 16 rounds of four halvings each took 7.6 us at 128 bins, and a search that falls
# back to equal steps alone takes as many.  Where every other round is a secant's, two of them gain at least 8 bits (6 beyond 512
# bins) before a bracket without kinks ends it: 11 rounds and 14 are the most of 1,500 score buffers.
@pytest.mark.parametrize("B,most", [(64, 11), (128, 11), (256, 11), (512, 11), (513, 14), (1024, 14), (2048, 14)])
def test_score_buffers_take_few_rounds(B, most):
    rng = np.random.default_rng(B)
    for kappa in (0.25, 0.5, 0.625):
        for M in (512, 4096, 32768, 262144):
            for _ in range(3):
                right = rng.random(M) < 0.4
                score = 1 / (1 + np.exp(-(rng.normal(size=M) + np.where(right, 0.8, -0.8))))
                b = np.minimum(B - 1, (score * B).astype(int))
                c_pos, c_neg = np.bincount(b[right], minlength=B), np.bincount(b[~right], minlength=B)
                args = (kappa, 0.5, 0.5, 0.05, 0.95, 1.0)
                rounds, delta = search(c_pos, c_neg, args)
                assert rounds <= most, (kappa, M)
                # both end at neighbouring doubles of the root; sums of B terms differ by B * 1.1e-16 over a slope of at least 1e-2
                assert abs(delta - O.calibrate(c_pos, c_neg, *(f32(x) for x in args))[2]) <= B * 1.1e-16 * 100 + 1e-15


# whatever the policy: four rounds of the secant's kind at most, 16 (21) of equal steps
@pytest.mark.parametrize("B,most", [(1, 20), (2, 20), (512, 20), (513, 25), (2048, 25)])
def test_rounds_are_bounded(B, most):
    rng = np.random.default_rng(B)
    for i in range(200):
        p_min, p_max = 0.5 * rng.random(), 1 - 0.5 * rng.random()
        args = (rng.random(), rng.random(), 10 ** rng.uniform(-3, 4), p_min, p_max, rng.choice([0.0, 0.01, 1.0]))
        counts = rng.integers(0, int(2 ** rng.uniform(1, 12)), (2, B))
        assert search(counts[0], counts[1], args)[0] <= most, (i, args)


def test_bad_arguments():
    c, out = np.zeros(4, np.int64), ctypes.create_string_buffer(8)
    ok = A.Policy(0.5, 0.5, 0.5, 0.05, 0.95, 1.0)
    call = lambda cp, B, pol, o: A.lib().arrol_calibrate_search(cp, c.ctypes.data, B, pol, o, out)
    assert call(c.ctypes.data, 4, ok, out) == 0
    for bad in ((None, 4, ok, out), (c.ctypes.data, 0, ok, out), (c.ctypes.data, 2049, ok, out), (c.ctypes.data, 4, A.Policy(2.0, 0.5, 0.5, 0.0, 1.0, 1.0), out),
                (c.ctypes.data, 4, ok, None)):
        assert call(*bad) == -1
