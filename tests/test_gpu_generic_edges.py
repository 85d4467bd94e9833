"""The scoring kernels for any shape against the fp64 oracle at the sizes where they change course: head dims around the
register classes (64, 128, 256), windows around the padded ones (8, 16, 32, 64), row counts that do and do not fit LDS
at once, lengths around a wavefront's and a workgroup's keys, chunk partials folded in either place."""

import numpy as np
import pytest

import gpu_helpers as H
from paper_2510_22556_amd import synth
from test_gpu_parity import torch_cuda  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("G,W,D,L,dtype", [
    (1, 1, 8, 33, "f32"), (3, 5, 16, 129, "f32"), (1, 8, 64, 31, "f32"), (4, 9, 72, 127, "f32"), (2, 16, 128, 128, "f32"),
    (7, 17, 136, 161, "f32"), (1, 33, 256, 1000, "f32"), (5, 64, 128, 257, "f32"), (8, 32, 256, 300, "f32"),
    (16, 64, 256, 200, "f32"), (200, 5, 24, 70, "f32"), (4, 32, 128, 9001, "f32"), (3, 12, 80, 515, "bf16"),
    (9, 16, 128, 2049, "bf16"), (5, 64, 256, 130, "bf16"), (2, 3, 256, 65, "bf16"),
])
def test_generic_scores_at_the_edges(oracle, torch_cuda, G, W, D, L, dtype):  # noqa: F811
    torch = torch_cuda
    from paper_2510_22556_amd import binding as B

    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    Hkv, seed = 2, G * 1000 + W + D + L
    q = synth.normal_torch(seed, 1, (1, 1, G * Hkv, W, D), "cuda", dt)
    k = synth.normal_torch(seed, 2, (1, 1, Hkv, L, 2 * D), "cuda", dt)[..., D:]          # rows farther apart than they are long
    shape = B.make_shape(q, k)
    ws = torch.empty((B.sablock_workspace_bytes(shape, 0, 0),), dtype=torch.uint8, device="cuda")
    s = torch.full((Hkv, L), float("nan"), dtype=torch.float32, device="cuda")
    e = torch.full_like(s, float("nan"))
    B.sablock_score(shape, q, k, s, e, ws)
    # the rows' denominators handed over: in fp64, rounded once
    x = (q[0, 0].view(Hkv, G * W, D).cpu().double() @ k[0, 0].cpu().double().transpose(1, 2)) / np.sqrt(D)
    t, i = torch.arange(L)[None, :], torch.arange(G * W)[:, None] % W
    x.masked_fill_((t > L - W + i)[None], float("-inf"))
    lse = torch.logsumexp(x, dim=2).float().view(1, 1, Hkv * G, W).cuda()
    s2, e2 = torch.full_like(s, float("nan")), torch.full_like(s, float("nan"))
    B.sablock_score(shape, q, k, s2, e2, ws, row_lse=lse)
    torch.cuda.synchronize()
    for p in range(Hkv):
        sr, er = oracle.score(H.widen(H.to_np(q[0, 0, p * G:(p + 1) * G].contiguous())), H.widen(H.to_np(k[0, 0, p].contiguous())), 1e-6)
        for a, b in ((s, e), (s2, e2)):
            # a D-term fp32 dot of unit normals is off by about sqrt(D) 2^-24 absolute, a probability by that relative
            np.testing.assert_allclose(H.to_np(a[p]), sr, rtol=1e-5, atol=1e-9)
            np.testing.assert_allclose(H.to_np(b[p]), er, rtol=1e-5, atol=2e-6)


@pytest.mark.parametrize("G,W,D,L,dtype", [(4, 16, 64, 3001, "f32"), (2, 64, 256, 700, "f32"), (4, 12, 80, 3001, "bf16"), (1, 1, 8, 70, "f32")])
@pytest.mark.parametrize("step", [17, 1000])
def test_generic_keys_that_are_not_numbers_are_no_part_of_the_others_denominators(torch_cuda, G, W, D, L, dtype, step):  # noqa: F811
    # their own score is not a number and their entropy term zero; every other key has the score it has without them
    torch = torch_cuda
    from paper_2510_22556_amd import binding as B

    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    q = synth.normal_torch(D + L, 1, (1, 1, G * 2, W, D), "cuda", dt)
    k = synth.normal_torch(D + L, 2, (1, 1, 2, L, D), "cuda", dt)
    bad = torch.zeros((L,), dtype=torch.bool, device="cuda")
    bad[::step] = True
    bad[min(L - 1, 64):min(L - 1, 128)] = True                 # whole tiles of them
    k[0, 0, 0, bad, 3] = float("nan")
    shape = B.make_shape(q, k)
    ws = torch.empty((B.sablock_workspace_bytes(shape, 0, 0),), dtype=torch.uint8, device="cuda")
    s = torch.empty((2, L), dtype=torch.float32, device="cuda")
    e = torch.empty_like(s)
    B.sablock_score(shape, q, k, s, e, ws)
    x = (q[0, 0, :G].reshape(G * W, D).double() @ k[0, 0, 0].double().T) / D ** 0.5
    t, i = torch.arange(L, device="cuda")[None, :], torch.arange(G * W, device="cuda")[:, None] % W
    x.masked_fill_((t > L - W + i) | bad[None, :], float("-inf"))
    ref = torch.softmax(x, dim=1).sum(dim=0) / G
    ok = ~bad
    assert torch.isnan(s[0, bad][:-W]).all() and (e[0, bad] == 0).all()
    np.testing.assert_allclose(s[0, ok].cpu().numpy(), ref[ok].cpu().numpy(), rtol=1e-5, atol=1e-9)
    assert torch.isfinite(e[0, ok]).all() and torch.isfinite(s[1]).all() and torch.isfinite(e[1]).all()
    # an infinite logit leaves no score of its rows
    k[0, 0, 0, bad, 3] = 0.0
    k[0, 0, 0, 2, 3] = float("inf")
    B.sablock_score(shape, q, k, s, e, ws)
    if (q[0, 0, :G, :, 3] > 0).any():
        assert not torch.isfinite(s[0, :L - W]).any()


@pytest.mark.parametrize("n_layers,Hkv,G,W,D,L", [(626, 64, 1, 8, 8, 150), (512, 16, 5, 1, 16, 300), (3, 2, 3, 5, 16, 4000)])
def test_generic_statistics_take_no_scratch_for_padding(torch_cuda, n_layers, Hkv, G, W, D, L):  # noqa: F811
    # 8 bytes per row and chunk of keys, whatever a window is padded to: calls of many problems fit the static array
    torch = torch_cuda
    from paper_2510_22556_amd import binding as B

    q = synth.normal_torch(L, 1, (1, n_layers, G * Hkv, W, D), "cuda", torch.float32)
    k = synth.normal_torch(L, 2, (1, n_layers, Hkv, L, D), "cuda", torch.float32)
    shape = B.make_shape(q, k)
    P = n_layers * Hkv
    need = B.sablock_workspace_bytes(shape, 0, 0)
    assert need <= 8 * P * G * W * (min(64, -(-L // 128)) + 1) + 256           # chunks of 128 keys or more, and their fold
    ws = torch.empty((need,), dtype=torch.uint8, device="cuda")
    out = [torch.full((P, L), float("nan"), device="cuda") for _ in range(4)]
    B.sablock_score(shape, q, k, out[0], out[1], ws)
    B.sablock_score_static(shape, q, k, out[2], out[3])
    torch.cuda.synchronize()
    assert torch.equal(out[0], out[2]) and torch.equal(out[1], out[3])
    p = P - 1
    x = (q[0, -1, -G:].reshape(G * W, D).double() @ k[0, -1, -1].double().T) / D ** 0.5
    t, i = torch.arange(L, device="cuda")[None, :], torch.arange(G * W, device="cuda")[:, None] % W
    x.masked_fill_(t > L - W + i, float("-inf"))
    ref = torch.softmax(x, dim=1).sum(dim=0) / G
    np.testing.assert_allclose(out[0][p].cpu().numpy(), ref.cpu().numpy(), rtol=1e-5, atol=1e-9)
