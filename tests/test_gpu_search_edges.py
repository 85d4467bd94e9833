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


def _scores(rng, kind, T):
    if kind == "smooth":                                       # sums that cannot round in segments of any length here
        return 1.0 + rng.random((2, T))
    if kind == "wide":                                         # sums that do
        return np.exp(5.0 * rng.standard_normal((2, T))) * 1e-6
    if kind == "levels":                                       # equal block sums by the hundred
        return np.round(rng.random((2, T)) ** 2 * 4) / 4
    return np.full((2, T), 0.25)                               # all of them


@pytest.mark.parametrize("n", [513, 640, 831, 833, 2047, 4097, 8193, 20000])
@pytest.mark.parametrize("kind", ["smooth", "wide", "levels", "equal"])
def test_search_and_selection_of_long_segments(oracle, torch_cuda, n, kind):  # noqa: F811
    # segments that are searched and selected from memory: block sums that are kept in LDS or formed in every pass, few
    # and many candidates for the last block, equal sums at the threshold; short last blocks; budgets that take a few
    # blocks, half of them, nearly all
    rng = np.random.default_rng(n)
    T = 2 * n + 77
    st = _scores(rng, kind, T)
    off = np.array([0, n, n + 70, 2 * n + 70, T], np.int32)
    for cand, budget, tau in (([1, 2, 3, 5, 8, 16, 31, 64], T // 50 + 2, 0.85), ([1, 2], T // 2, 0.9999), ([1, 3, 64], T - 3, 1.0),
                              ([1, 7, 33], 130, 0.2), ([1, 2, 64], T // 3, 1.5)):
        _assert_search_select(oracle, torch_cuda, st, off, cand, budget, tau)


@pytest.mark.parametrize("n", [64, 300, 512, 513, 4096, 4097, 9001])
@pytest.mark.parametrize("g", [1, 2, 3, 64])
def test_selection_with_a_caller_s_own_budgets(oracle, torch_cuda, n, g):  # noqa: F811
    # b_k and g_k* that no search gave: tokens ranked (g = 1) and blocks filled at lengths each side of every layout
    torch = torch_cuda
    from paper_2510_22556_amd import binding as B
    from test_gpu_parity import _stage_inputs

    rng = np.random.default_rng(n + g)
    off = np.array([0, n, n + 5, 2 * n + 5], np.int32)
    T = int(off[-1])
    st = np.round(rng.random((2, T)) * 500) / 512
    bk = np.array([max(n // 3, g), 2, max(n - 1, g)], np.int32)               # a block size is at most b_k
    gs = np.array([g, 1, g], np.int32)
    budget = int(bk.sum())
    q, k = _stage_inputs(torch, st)
    shape, seg = B.make_shape(q, k), B.make_segments(off, [0, len(off)], "cuda")
    buf = B.Buffers(shape, seg, budget, "cuda")
    d = {x: torch.as_tensor(np.tile(y, (2, 1))).cuda() for x, y in (("b", bk), ("g", gs))}
    B.sablock_select(shape, torch.as_tensor(st.astype(np.float32)).cuda(), seg, d["b"], d["g"], budget, buf.idx, buf.n_sel, buf.ws)
    torch.cuda.synchronize()
    for p in range(2):
        idx, n_sel = oracle.select(st[p].astype(np.float32), off, bk, gs, budget)
        assert int(buf.n_sel[p]) == n_sel == budget
        np.testing.assert_array_equal(buf.idx[p].cpu().numpy(), idx)


@pytest.mark.parametrize("kind", ["smooth", "wide"])
def test_a_long_segment_does_not_hold_up_the_call(torch_cuda, kind):  # noqa: F811
    # one segment of 16 384 tokens among short ones: 6 and 9 times the call without it where the blocks taken are found by
    # their sums, 20 000 times where every block is ranked against every other with sums formed again for each pair
    torch = torch_cuda
    from paper_2510_22556_amd import binding as B

    T, P, W, budget = 131040, 8, 32, 992
    rng = np.random.default_rng(5)
    q = torch.zeros((1, P, 1, W, 8), dtype=torch.float32, device="cuda")
    shape = B.make_shape(q, torch.zeros((1, P, 1, T + W, 8), dtype=torch.float32, device="cuda"))
    st = torch.as_tensor(np.tile(_scores(rng, kind, T), (P // 2, 1)).astype(np.float32)).cuda()
    us = []
    for first in (48, 16384):
        off = np.unique(np.concatenate([[0], np.arange(first, T, 48), [T]]))
        seg = B.make_segments(off, [0, len(off)], "cuda")
        buf = B.Buffers(shape, seg, budget, "cuda")
        times = []
        for _ in range(4):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            B.sablock_search_select(shape, st, seg, [1, 8, 16, 32, 64], budget, 0.85, buf.seg_budget, buf.block_size, buf.idx, buf.n_sel, buf.ws)
            b.record()
            torch.cuda.synchronize()
            times.append(a.elapsed_time(b) * 1e3)
        us.append(min(times))
    assert us[1] < 100 * us[0], us


@pytest.mark.parametrize("T", [1023, 16385, 40001])
@pytest.mark.parametrize("budget", [100, 3000, 6000])
def test_topb_with_more_rows_than_compute_units(oracle, torch_cuda, T, budget):  # noqa: F811
    # two workgroups per compute unit: the kernels with fewer registers, for lists of 4 096 and 8 192 tokens
    rng = np.random.default_rng(T)
    st = rng.random((3, T)) ** 4
    off = _offsets(rng, T, rng.integers(1, 80, size=T))
    _assert_search_select(oracle, torch_cuda, st, off, CAND, min(budget, T - 1), 0.85, compute_units=2)


@pytest.mark.parametrize("T", [5000, 20000, 40001])
@pytest.mark.parametrize("sign", [1, -1])
def test_scores_that_are_not_numbers_rank_alike_in_rows_of_every_length(torch_cuda, T, sign):  # noqa: F811
    # by their bits, in front of every number or behind: the Top-B tokens, the budgets and the tokens written agree,
    # however the k-th best is found
    rng = np.random.default_rng(T)
    st = rng.random((2, T)).astype(np.float32)
    bits = st.view(np.uint32)
    bits[:, rng.permutation(T)[:40]] = 0x7FC00000 if sign > 0 else 0xFFC00000
    bits[:, T - 1] = bits[:, 0] = 0x7FC00001                   # the scalars around the row's vectors
    key = np.where(bits >> 31, ~bits, bits | 0x80000000).astype(np.int64)
    off = _offsets(rng, T, rng.integers(1, 80, size=T))
    for budget in (3, 100, 900):
        from test_gpu_parity import _search_select_gpu

        b, g, idx, n = _search_select_gpu(torch_cuda, st, off, [1], budget, 0.85)
        for p in range(2):
            best = np.sort(np.lexsort((np.arange(T), -key[p]))[:budget])
            assert n[p] == budget
            np.testing.assert_array_equal(idx[p][:budget], best)
            np.testing.assert_array_equal(b[p][:len(off) - 1], np.diff(np.searchsorted(best, off)))


@pytest.mark.parametrize("n", [64, 300, 513, 4096, 9001])
@pytest.mark.parametrize("share", [0.02, 0.5, 1.0])
def test_scores_that_are_not_numbers_take_a_segment_s_share_and_no_more(torch_cuda, n, share):  # noqa: F811
    # every segment gives its b_k tokens, ascending and its own, whichever blocks and tokens those are: with given block
    # sizes (few and many blocks taken, blocks cut) and through the search
    torch = torch_cuda
    from paper_2510_22556_amd import binding as B
    from test_gpu_parity import _search_select_gpu, _stage_inputs

    rng = np.random.default_rng(n)
    off = np.array([0, n, n + 5, 2 * n + 5], np.int32)
    T = int(off[-1])
    st = rng.random((2, T)).astype(np.float32)
    st[rng.random((2, T)) < share] = np.nan
    st[1] = -st[1]
    tokens = torch.as_tensor(st).cuda()
    q, k = _stage_inputs(torch, st)
    shape, seg = B.make_shape(q, k), B.make_segments(off, [0, len(off)], "cuda")

    def check(idx, b):
        for p in range(2):
            assert (np.diff(idx[p]) > 0).all() and idx[p][0] >= 0 and idx[p][-1] < T
            np.testing.assert_array_equal(np.diff(np.searchsorted(idx[p], off)), b[p])

    for g in (1, 2, 7, 64):
        for bk in ([max(g, 3), 2, max(n // 2, g)], [max(n // 3, g), 3, n - 1 if g < n else n]):
            budget = sum(bk)
            buf = B.Buffers(shape, seg, budget, "cuda")
            d = [torch.as_tensor(np.tile(np.array(x, np.int32), (2, 1))).cuda() for x in (bk, [g, 1, g])]
            B.sablock_select(shape, tokens, seg, *d, budget, buf.idx, buf.n_sel, buf.ws)
            check(buf.idx.cpu().numpy(), [bk, bk])
    for budget in (7, T // 3, T - 2):
        b, g, idx, _ = _search_select_gpu(torch, st, off, [1, 2, 3, 8, 64], budget, 0.85)
        check(idx[:, :budget], b[:, :len(off) - 1])


@pytest.mark.parametrize("T", [1, 255, 4096, 4097, 8192, 8193, 16384])
@pytest.mark.parametrize("mean", [1, 2, 30])
@pytest.mark.parametrize("levels", [0, 3])
def test_rows_and_segments_around_the_threads_that_hold_them(oracle, torch_cuda, T, mean, levels):  # noqa: F811
    # 256, 512 or 1 024 threads by the row's length; more segments than threads, as many as tokens (mean 1);
    # levels: more ties at the threshold than are ranked, cut by index
    rng = np.random.default_rng(T + mean)
    st = rng.random((3, T)) ** 3
    if levels:
        st = np.round(st * levels) / levels
    off = _offsets(rng, T, rng.integers(1, 2 * mean, size=T) if mean > 1 else np.ones(T, np.int64))
    for budget in sorted({1, T // 7, T // 2, T - 1} - {0}):
        _assert_search_select(oracle, torch_cuda, st, off, CAND, budget, 0.85)


@pytest.mark.parametrize("T", [2049, 4096, 8161, 16000])
@pytest.mark.parametrize("cus", [2, 256])
@pytest.mark.parametrize("levels", [0, 3])
def test_rows_around_the_number_of_segments_that_changes_their_kernel(oracle, torch_cuda, T, cus, levels):  # noqa: F811
    # half as many segments as tokens, three quarters, what two workgroups have room for; rows beyond the compute units and not
    rng = np.random.default_rng(T + cus)
    st = rng.random((3, T)) ** 3
    if levels:
        st = np.round(st * levels) / levels
    for n in {min(n, T) for n in (2048, 2049, T // 2, T // 2 + 1, T // 4 * 3, T // 4 * 3 + 1, 5300, 5400)}:
        off = np.concatenate([[0], np.sort(rng.choice(T - 1, n - 1, replace=False)) + 1, [T]]).astype(np.int32)
        for budget in (T // 9, T // 2):
            _assert_search_select(oracle, torch_cuda, st, off, CAND, budget, 0.85, compute_units=cus)


@pytest.mark.parametrize("levels", [0, 3])
def test_listed_rows_of_as_many_segments_as_one_call_takes(oracle, torch_cuda, levels):  # noqa: F811
    # long rows whose better tokens are listed by several workgroups (levels: more ties than the lists hold), ranked by 512 threads, by
    # 1 024, and by the kernel for any number of segments
    rng = np.random.default_rng(levels)
    T = 131072
    st = rng.random((3, T)) ** 5
    if levels:
        st = np.round(st * levels) / levels
    for n in (2048, 2049, 11431, 11432, 16383):
        off = np.concatenate([[0], np.sort(rng.choice(T - 1, n - 1, replace=False)) + 1, [T]]).astype(np.int32)
        for budget in (700, 2000):
            _assert_search_select(oracle, torch_cuda, st, off, CAND, budget, 0.85)
