"""Decode attention at the sizes where its kernels change course, against the fp64 oracle: every group size, row widths from
4 to 64 lanes, one split and many, splits that hold no entry at all, references that have to move."""

import numpy as np
import pytest

import gpu_helpers as H
from paper_2510_22556_amd import synth
from test_gpu_parity import torch_cuda  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("G,D,dtype", [(1, 32, "bf16"), (2, 64, "bf16"), (3, 128, "bf16"), (5, 32, "bf16"), (8, 64, "bf16"),
                                       (8, 128, "bf16"), (4, 256, "bf16"), (6, 16, "f32"), (7, 64, "f32"), (8, 128, "f32"), (4, 256, "f32")])
@pytest.mark.parametrize("rows,n_sel", [(2, None), (129, 1), (256, None), (257, 0), (2048, 700), (5000, 0), (40000, None)])
def test_decode_group_sizes_rows_and_splits(oracle, torch_cuda, G, D, dtype, rows, n_sel):  # noqa: F811
    torch = torch_cuda
    from paper_2510_22556_amd import binding as B

    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    P, seed = 2, G * 1000 + D + rows
    q = synth.normal_torch(seed, 1, (1, 1, G * P, D), "cuda", dt)
    k = synth.normal_torch(seed, 2, (1, 1, P, rows, D), "cuda", dt)
    v = synth.normal_torch(seed, 3, (1, 1, P, rows, D), "cuda", dt)
    k[0, 0, 0, -1] = (q[0, 0, G - 1].float() * (120.0 / D ** 0.5)).to(dt)      # a late logit far ahead of the others
    budget = rows - 2
    sel = None if n_sel is None else torch.tensor([n_sel, min(n_sel + 1, budget)], dtype=torch.int32, device="cuda")
    shape = B.make_cache_shape(q, k, v)
    ws = torch.full((B.sablock_decode_workspace_bytes(shape),), 0xFF, dtype=torch.uint8, device="cuda")
    out = torch.full(q.shape, float("nan"), dtype=torch.float32, device="cuda")
    B.sablock_decode_attention(shape, q, k, v, out, ws, n_sel=sel, budget=budget if sel is not None else 0)
    torch.cuda.synchronize()
    for p in range(P):
        keep = np.arange(rows)
        if sel is not None:
            keep = keep[(keep < int(sel[p])) | (keep >= budget)]
        ref = oracle.decode_attention(H.widen(H.to_np(q[0, 0, p * G:(p + 1) * G])), H.widen(H.to_np(k[0, 0, p]))[keep],
                                      H.widen(H.to_np(v[0, 0, p]))[keep])
        # fp32 logits of magnitude <= 250 in the log2 domain: 2^-17 relative in a probability
        np.testing.assert_allclose(H.to_np(out[0, 0, p * G:(p + 1) * G]), ref, rtol=2e-5, atol=4e-5)
