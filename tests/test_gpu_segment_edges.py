"""Segmentation at the sizes where its kernels change course (steps of 256 tokens, four in flight, sixteen wavefronts, up to
eight slices, masks too many for LDS), rows at every alignment, delimiters at every place: whole numbers, exact."""

import ctypes

import numpy as np
import pytest

from test_gpu_parity import torch_cuda  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T", [1, 2, 3, 255, 256, 257, 4096, 4099, 16383, 16384, 65472, 131075, 4_200_001])
@pytest.mark.parametrize("density,delims", [(0.0, [7]), (0.02, [5, 9, -1]), (1.0, [1, 2]), (0.3, list(range(64))), (0.5, []), (0.02, [5.0, 9.0])])
def test_segment_offsets_at_the_edges(oracle, torch_cuda, T, density, delims):  # noqa: F811
    torch = torch_cuda
    from paper_2510_22556_amd import binding as B

    density = min(density, 0.02) if T > 1_000_000 else density
    rng = np.random.default_rng(T)
    n_seq = 2 if T > 1_000_000 else 3
    tok = rng.integers(1000, 2000, size=(n_seq, T + 3)).astype(np.int32)
    if delims:
        hit = rng.random(tok.shape) < density
        tok[hit] = rng.choice(delims, size=int(hit.sum()))
    dev = torch.as_tensor(tok).cuda()[:, 1:T + 1]              # rows start at any token, three beyond their end belong to others
    seg = B.segment(dev, delims)
    off = seg.seg_off.cpu().numpy()
    for s in range(n_seq):
        ref = oracle.segment(tok[s, 1:T + 1], delims) if T < 1_000_000 else np.concatenate(
            [[0], np.flatnonzero(np.isin(tok[s, 1:T], delims)) + 1, [T]])
        np.testing.assert_array_equal(off[seg.seg_ptr[s]:seg.seg_ptr[s + 1]], ref)


def test_segment_whatever_torch_s_default_device_is(torch_cuda):  # noqa: F811
    # the counts go to pinned host memory, which a program that creates its tensors on the GPU by default has to get too
    torch = torch_cuda
    from paper_2510_22556_amd import binding as B

    tok = torch.full((2, 100), 1000, dtype=torch.int32, device="cuda")
    tok[0, 9] = tok[1, 19] = tok[1, 29] = 7
    before = torch.get_default_device()
    torch.set_default_device("cuda")
    try:
        seg = B.segment(tok, [7])
    finally:
        torch.set_default_device(before if before.type != "cpu" else None)
    assert seg.seg_off.cpu().tolist() == [0, 10, 100, 0, 20, 30, 100] and list(seg.seg_ptr) == [0, 3, 7]


def _tokens(torch, T, n_seq=2):
    tok = np.random.default_rng(T).integers(0, 40, size=(n_seq, T)).astype(np.int32)
    return tok, torch.as_tensor(tok).cuda()


@pytest.mark.parametrize("T", [1, 257, 4099, 16384, 65472, 131075])
def test_the_calls_by_whole_sequences_give_the_same(oracle, torch_cuda, T):  # noqa: F811
    torch = torch_cuda
    from paper_2510_22556_amd import binding as B

    tok, dev = _tokens(torch, T)
    ref = [oracle.segment(row, [3, 5]) for row in tok]
    seg = B.segment(dev, [3, 5])
    count = torch.empty((2,), dtype=torch.int32, device="cuda")
    B.sablock_segment_count(dev, [3, 5], count)
    ptr = [0] + [int(x) for x in np.cumsum(count.cpu().numpy() + 1)]
    off = torch.full((ptr[-1],), -1, dtype=torch.int32, device="cuda")
    B.sablock_segment_offsets(dev, [3, 5], ptr, off)
    assert ptr == list(seg.seg_ptr) and torch.equal(off, seg.seg_off)
    np.testing.assert_array_equal(off.cpu().numpy(), np.concatenate(ref))


@pytest.mark.parametrize("T", [1, 257, 4099, 16383, 16384, 16385, 32768, 65472, 131075])
@pytest.mark.parametrize("short", [0, 3])
def test_the_calls_by_slices(oracle, torch_cuda, T, short):  # noqa: F811
    # one slice and several, the last one of a token, a step or full; with `short` places too few for the last slice: its last
    # boundaries are dropped, both ends are written, and nothing is outside the room that the places leave
    torch = torch_cuda
    from paper_2510_22556_amd import binding as B

    lib, n_seq = B.load(), 2
    tok, dev = _tokens(torch, T, n_seq)
    delims, st = (ctypes.c_int32 * 2)(3, 5), torch.cuda.current_stream().cuda_stream or None
    per = lib.sablock_segment_slices(n_seq, T)
    assert per == -(-T // B.SLICE_TOKENS)
    count = torch.full((n_seq * per,), -1, dtype=torch.int32, device="cuda")
    args = (dev.data_ptr(), T, n_seq, T, delims, 2)
    assert lib.sablock_segment_slice_count(*args, count.data_ptr(), st) == 0
    ref = [oracle.segment(row, [3, 5]) for row in tok]
    inner = [r[1:-1] for r in ref]
    at = count.cpu().numpy().reshape(n_seq, per)
    for s in range(n_seq):                                     # a boundary belongs to the slice of the delimiter in front of it
        np.testing.assert_array_equal(at[s], np.bincount((inner[s] - 1) // B.SLICE_TOKENS, minlength=per))
    short = min(short, int(at[-1, -1]))
    place = [4]                                                # the offsets begin behind a few words of others
    for s in range(n_seq):
        for i in range(per):
            place.append(place[-1] + int(at[s, i]) + (2 if i == per - 1 else 0))
    place[-1] -= short
    off = torch.full((place[-1] + 64,), -7, dtype=torch.int32, device="cuda")
    assert lib.sablock_segment_slice_offsets(*args, (ctypes.c_int32 * len(place))(*place), off.data_ptr(), st) == 0
    want = np.full(place[-1] + 64, -7, dtype=np.int32)
    want[4:4 + len(ref[0])] = ref[0]
    last = ref[1] if short == 0 else np.concatenate([ref[1][:-1 - short], [T]])
    want[4 + len(ref[0]):place[-1]] = last
    np.testing.assert_array_equal(off.cpu().numpy(), want)
