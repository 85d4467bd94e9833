"""Row statistics of the matrix-pipe scoring kernels against the fp64 oracle where their loop changes course: a row's
reference moved in each tile of rows (the one left waiting under the next subtile among them), streams of one subtile,
first subtiles that touch the window, prompts shorter than a workgroup's stride."""

import numpy as np
import pytest

import gpu_helpers as H
from paper_2510_22556_amd import synth
from test_gpu_parity import torch_cuda  # noqa: F401

pytestmark = pytest.mark.gpu

SHAPES = [(4, 32, 128), (7, 16, 128), (3, 32, 128), (5, 8, 128), (1, 8, 128), (2, 64, 128), (4, 32, 64), (3, 32, 96), (2, 32, 256), (3, 32, 256)]


def _check(oracle, torch, q, k, Hkv, G, W, D, L, **tuning):
    from paper_2510_22556_amd import binding as B

    shape = B.make_shape(q, k, **tuning)
    ws = torch.empty((B.sablock_workspace_bytes(shape, 0, 0),), dtype=torch.uint8, device="cuda")
    s = torch.full((Hkv, L), float("nan"), dtype=torch.float32, device="cuda")
    e = torch.full_like(s, float("nan"))
    B.sablock_score(shape, q, k, s, e, ws)
    torch.cuda.synchronize()
    for p in range(Hkv):
        sr, er = oracle.score(H.widen(H.to_np(q[0, 0, p * G:(p + 1) * G].contiguous())), H.widen(H.to_np(k[0, 0, p].contiguous())), 1e-6)
        # a logit of up to 300 in the log2 domain is rounded to 2^-16 in fp32, a probability by that relative
        np.testing.assert_allclose(H.to_np(s[p]), sr, rtol=5e-5, atol=1e-9)
        np.testing.assert_allclose(H.to_np(e[p]), er, rtol=5e-5, atol=5e-6)


@pytest.mark.parametrize("G,W,D", SHAPES)
def test_a_reference_moves_in_every_tile(oracle, torch_cuda, G, W, D):  # noqa: F811
    torch = torch_cuda
    Hkv, L = 2, 4096 + 45 + W
    q = synth.normal_torch(G * W + D, 1, (1, 1, G * Hkv, W, D), "cuda", torch.bfloat16)
    k = synth.normal_torch(G * W + D, 2, (1, 1, Hkv, L, D), "cuda", torch.bfloat16)
    at = 130                                    # 32 keys to a subtile, every fourth subtile to one wavefront
    for r in list(range(0, G * W, 32)) + [G * W - 1]:
        for p in range(Hkv):
            row = q[0, 0, p * G + r // W, r % W].float()
            for t, scale in ((at, 5.0), (at + 128 * (1 + p), 9.0), (at + 1024, 12.0)):
                k[0, 0, p, t] = (row * scale * (128 / D) ** 0.5).to(torch.bfloat16)
        at += 301
    _check(oracle, torch, q, k, Hkv, G, W, D, L, score_chunk=1024)


@pytest.mark.parametrize("G,W,D", SHAPES)
@pytest.mark.parametrize("T", [1, 31, 32, 33, 64, 127, 129, 160])
def test_short_streams(oracle, torch_cuda, G, W, D, T):  # noqa: F811
    torch = torch_cuda
    q = synth.normal_torch(T, 1, (1, 1, G * 2, W, D), "cuda", torch.bfloat16)
    k = synth.normal_torch(T, 2, (1, 1, 2, T + W, D), "cuda", torch.bfloat16)
    _check(oracle, torch, q, k, 2, G, W, D, T + W, score_chunk=128)


@pytest.mark.parametrize("G,W,D", SHAPES + [(8, 32, 128), (4, 64, 128)])
@pytest.mark.parametrize("logit", [-120.0, 60.0, 95.0])
def test_rows_whose_logits_lie_far_from_zero(oracle, torch_cuda, G, W, D, logit):  # noqa: F811
    # sums that under- or overflow without a reference, in one row of every head: those wavefronts start again with one
    torch = torch_cuda
    Hkv, L = 2, 1024 + 45 + W
    q = synth.normal_torch(G * W + D, 3, (1, 1, G * Hkv, W, D), "cuda", torch.bfloat16)
    k = synth.normal_torch(G * W + D, 4, (1, 1, Hkv, L, D), "cuda", torch.bfloat16)
    k[..., 0] = 1.0
    q[:, :, :, W // 2, 0] = logit * D ** 0.5                   # every logit of the row moves by that much
    _check(oracle, torch, q, k, Hkv, G, W, D, L, score_chunk=512)
