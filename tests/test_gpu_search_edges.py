"""Search and selection at the sizes where their kernels change course, bit for bit against the fp64 oracle.

The Top-B kernel holds rows of up to 16 384 tokens in registers and bounds longer ones by a sample; the search keeps
prefix sums where no sum of a segment's scores can round and orders its sums otherwise.
"""

import numpy as np
import pytest

from test_gpu_parity import _assert_search_select, torch_cuda  # noqa: F401

pytestmark = pytest.mark.gpu
CAND = [1, 2, 3, 4, 8, 16, 31, 64]


def _offsets(rng, T, lens):
    return np.unique(np.minimum(np.concatenate([[0], np.cumsum(lens)]), T)).astype(np.int32)


@pytest.mark.parametrize("T", [1, 3, 1023, 16383, 16384, 16385, 16393, 40001])
@pytest.mark.parametrize("kind", ["smooth", "sorted", "late", "levels", "two"])
def test_topb_rows_around_the_register_round_and_samples_that_mislead(oracle, torch_cuda, T, kind):  # noqa: F811
    # sorted: the sample is exact in spirit; late: all the best tokens sit in 1 % of the row; levels / two: more ties at
    # the threshold than are ranked, or than the list holds.  Odd T: rows at every alignment.
    rng = np.random.default_rng(T)
    st = rng.random((3, T)) ** 4
    if kind == "sorted":
        st = np.sort(st, axis=1)
    elif kind == "late":
        st[:, T - max(T // 100, 1):] += 1.0
    elif kind == "levels":
        st = np.round(st * 8) / 8
    elif kind == "two":
        st = (rng.random((3, T)) < 0.5).astype(np.float64)
    off = _offsets(rng, T, rng.integers(1, 80, size=T))
    for budget in sorted({1, max(T // 40, 1), max(T // 3, 1), max(T - 1, 1)}):
        if budget <= T:
            _assert_search_select(oracle, torch_cuda, st, off, CAND, budget, 0.85)


@pytest.mark.parametrize("n", [2, 63, 64, 65, 127, 128, 129, 511, 512, 639, 640, 1023, 1024, 4095, 4096])
@pytest.mark.parametrize("spread", [0, 16, 24, 40])
def test_search_segment_lengths_and_score_ranges(oracle, torch_cuda, n, spread):  # noqa: F811
    # segments of one length each side of every change of layout; scores over 2^spread: sums that cannot round (0), that
    # do in the longer segments only (16), in all of them (24, 40)
    rng = np.random.default_rng(n + spread)
    n_seg = max(4, min(40, 6000 // n))
    T = n * n_seg + 5
    st = (1.0 + rng.random((2, T))) * 2.0 ** -rng.integers(0, spread + 1, size=(2, T))
    st[1, rng.random(T) < 0.3] = 0.0
    off = _offsets(rng, T, np.full(n_seg + 6, n))
    for budget, tau in ((T // 25 + 1, 0.85), (T // 3, 0.97), (T // 2, 0.3)):
        _assert_search_select(oracle, torch_cuda, st, off, CAND, budget, tau)
