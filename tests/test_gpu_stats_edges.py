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


def _check(oracle, torch, q, k, Hkv, G, W, D, L, all_heads=False, row_lse=None, **tuning):
    from paper_2510_22556_amd import binding as B

    shape = B.make_shape(q, k, **tuning)
    call, n_ws = ((B.sablock_score_all_heads, B.sablock_score_all_heads_workspace_bytes(shape)) if all_heads else
                  (B.sablock_score, B.sablock_workspace_bytes(shape, 0, 0)))
    ws = torch.empty((n_ws,), dtype=torch.uint8, device="cuda")
    s = torch.full((1 if all_heads else Hkv, L), float("nan"), dtype=torch.float32, device="cuda")
    e = torch.full_like(s, float("nan"))
    call(shape, q, k, s, e, ws, row_lse=row_lse)
    torch.cuda.synchronize()
    for p in range(len(s)):
        of = oracle.score_layer if all_heads else oracle.score
        qp, kp = (q[0, 0], k[0, 0]) if all_heads else (q[0, 0, p * G:(p + 1) * G], k[0, 0, p])
        sr, er = of(H.widen(H.to_np(qp.contiguous())), H.widen(H.to_np(kp.contiguous())), 1e-6)
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


FAR = SHAPES + [(7, 32, 128), (8, 32, 128), (4, 64, 128), (5, 16, 256), (6, 8, 256)]


# the all-head call takes up to 128 rows of heads of 128 elements and windows of up to 32
@pytest.mark.parametrize("entry,G,W,D", [(e, *f) for e in ("score", "row_lse") for f in FAR] +
                         [("all_heads", *f) for f in FAR if f[2] == 128 and f[1] <= 32 and f[0] * f[1] <= 128])
@pytest.mark.parametrize("rows,logit,sink", [("all", -100.0, 20.0), ("first", -100.0, 0.0), ("first", 60.0, 0.0), ("all", 60.0, 20.0)])
def test_probabilities_of_rows_far_from_zero_are_not_flushed(oracle, torch_cuda, G, W, D, rows, logit, sink, entry):  # noqa: F811
    # all rows, or the first row of every head alone, at a logit that the first element makes; one key `sink` above
    # the others, whose probabilities of 2^-29 and less are in fp32's range whatever the rows' log-sum-exps
    torch = torch_cuda
    Hkv, L = 8 if entry == "all_heads" else 2, 1024 + 45 + W
    q = synth.normal_torch(G * W + D, 5, (1, 1, G * Hkv, W, D), "cuda", torch.bfloat16)
    k = synth.normal_torch(G * W + D, 6, (1, 1, Hkv, L, D), "cuda", torch.bfloat16)
    k[..., 0] = 1.0
    k[:, :, :, 300, 0] = 1.0 + sink / logit
    q[:, :, :, slice(None) if rows == "all" else slice(0, 1), 0] = logit * D ** 0.5
    lse = None
    if entry == "row_lse":
        x = torch.matmul(q[0, 0].double().reshape(Hkv, G * W, D), k[0, 0].double().transpose(1, 2).contiguous()) / D ** 0.5
        seen = torch.arange(L, device="cuda")[None] <= L - W + torch.arange(W, device="cuda").repeat(G)[:, None]
        lse = torch.logsumexp(x.masked_fill(~seen, float("-inf")), -1).float().contiguous()
    _check(oracle, torch, q, k, Hkv, G, W, D, L, all_heads=entry == "all_heads", row_lse=lse, score_chunk=512)


@pytest.mark.parametrize("G,W,D", FAR + [(6, 32, 128), (3, 64, 128), (3, 16, 128)])
@pytest.mark.parametrize("logits", [(-60.0, -60.0), (80.0, 80.0), (0.0, 100.0), (-68.0, 0.0)])
def test_rows_far_from_zero_in_long_streams(oracle, torch_cuda, G, W, D, logits):  # noqa: F811
    # 33 subtiles to a stream.  All logits far from zero: a walk with references, begun after the first sixteen subtiles;
    # only those of the last third far from the first subtile's: references that have to move
    torch = torch_cuda
    Hkv, L = 2, 4096 + 77 + W
    q = synth.normal_torch(G * W + D, 7, (1, 1, G * Hkv, W, D), "cuda", torch.bfloat16)
    k = synth.normal_torch(G * W + D, 8, (1, 1, Hkv, L, D), "cuda", torch.bfloat16)
    q[..., 0] = D ** 0.5
    k[..., 0] = logits[0]
    k[:, :, :, 2800:, 0] = logits[1]
    _check(oracle, torch, q, k, Hkv, G, W, D, L, score_chunk=8192)


@pytest.mark.parametrize("G,W", [(4, 32), (4, 16), (7, 32), (4, 64)])
@pytest.mark.parametrize("logit", [-50.0, 80.0])
def test_rows_far_from_zero_cost_little_more(torch_cuda, G, W, logit):  # noqa: F811
    # sixteen of 64 subtiles a second time and the references of a tile and subtile from LDS: less than half of one pass in two,
    # where a walk of its own for every tile is three times the call and more
    torch = torch_cuda
    from paper_2510_22556_amd import binding as B

    Hkv, L, D = 32, 65536, 128
    q = synth.normal_torch(G * W, 9, (1, 1, G * Hkv, W, D), "cuda", torch.bfloat16)
    k = synth.normal_torch(G * W, 10, (1, 1, Hkv, L, D), "cuda", torch.bfloat16)
    q[..., 0] = D ** 0.5
    shape = B.make_shape(q, k)
    s = torch.empty((Hkv, L), dtype=torch.float32, device="cuda")
    e, ws = torch.empty_like(s), torch.empty((B.sablock_workspace_bytes(shape, 0, 0),), dtype=torch.uint8, device="cuda")

    def took():
        times = []
        for _ in range(15):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            B.sablock_score(shape, q, k, s, e, ws)
            b.record()
            b.synchronize()
            times.append(a.elapsed_time(b))
        return sorted(times)[7]

    k[..., 0] = 0.0
    near = took()
    k[..., 0] = logit
    assert took() < 1.5 * near


@pytest.mark.parametrize("G,W", [(1, 64), (2, 32), (4, 16), (4, 32), (7, 16)])
def test_peaked_rows_round_to_little(torch_cuda, G, W):  # noqa: F811
    # 64 keys scaled by four, scores against 64 bits: the exponents of a row's peak are small beside the row's reference.  Means
    # over eight heads and six seeds: 3.3e-7 to 4.4e-7, without references 6.0e-7 to 7.0e-7; the bound lies between
    torch = torch_cuda
    from paper_2510_22556_amd import binding as B

    Hkv, L, D, errors = 8, 1024, 128, []
    seen = torch.arange(L, device="cuda")[None] <= L - W + torch.arange(W, device="cuda").repeat(G)[:, None]
    for seed in range(6):
        gen = torch.Generator(device="cuda")
        gen.manual_seed(seed)
        q = torch.randn((1, 1, Hkv * G, W, D), generator=gen, device="cuda", dtype=torch.bfloat16)
        k = torch.randn((1, 1, Hkv, L, D), generator=gen, device="cuda", dtype=torch.bfloat16)
        k[:, :, :, torch.randperm(L - W, generator=gen, device="cuda")[:64]] *= 4.0
        shape = B.make_shape(q, k)
        s = torch.empty((Hkv, L), device="cuda")
        B.sablock_score(shape, q, k, s, torch.empty_like(s), torch.empty((B.sablock_workspace_bytes(shape, 0, 0),), dtype=torch.uint8, device="cuda"))
        x = torch.matmul(q[0, 0].double().reshape(Hkv, G * W, D), k[0, 0].double().transpose(1, 2).contiguous()) / D ** 0.5
        ref = torch.softmax(x.masked_fill(~seen, float("-inf")), -1).reshape(Hkv, G, W, L).mean(1).sum(1)
        errors.append(((s.double() - ref).norm(dim=1) / ref.norm(dim=1)).mean().item())
    assert sum(errors) / len(errors) < 5.2e-7


@pytest.mark.parametrize("cus", [1, 5, 9, 16, 20])
@pytest.mark.parametrize("Hkv,G,W,D,all_heads", [(7, 4, 32, 128, False), (3, 8, 32, 128, False), (5, 2, 8, 64, False), (8, 4, 32, 128, True)])
def test_chunks_of_a_plan_for_other_numbers_of_compute_units(oracle, torch_cuda, cus, Hkv, G, W, D, all_heads):  # noqa: F811
    # whole rounds of equal chunks, and larger ones with a shorter remainder (7 problems on 16 units: three to a problem)
    torch = torch_cuda
    L = 2900 + W
    q = synth.normal_torch(cus, 1, (1, 1, G * Hkv, W, D), "cuda", torch.bfloat16)
    k = synth.normal_torch(cus, 2, (1, 1, Hkv, L, D), "cuda", torch.bfloat16)
    _check(oracle, torch, q, k, Hkv, G, W, D, L, all_heads=all_heads, compute_units=cus)
    if D == 128:
        from paper_2510_22556_amd import binding as B

        def attend(**tuning):
            shape = B.make_shape(q, k, **tuning)
            out = torch.full((1, 1, G * Hkv, W, D), float("nan"), dtype=torch.float32, device="cuda")
            lse = torch.full((1, 1, G * Hkv, W), float("nan"), dtype=torch.float32, device="cuda")
            ws = torch.empty((B.sablock_window_attention_workspace_bytes(shape),), dtype=torch.uint8, device="cuda")
            B.sablock_window_attention(shape, q, k, k, out, lse, ws)
            return H.to_np(out), H.to_np(lse)

        (o, z), (o1, z1) = attend(compute_units=cus), attend(window_chunk=4096)
        # probabilities of either cut are rounded to bf16 by themselves, 2^-9 each; log-sum-exps are fp32
        np.testing.assert_allclose(z, z1, rtol=0, atol=2e-5)
        np.testing.assert_allclose(o, o1, rtol=0, atol=2e-3 * float(k.abs().max()))
