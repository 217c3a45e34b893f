"""hetis_attn_merge around the edges of its batches: 8 loads, 32 partial results, 64 log-sum-exps."""
import numpy as np
import pytest
import torch

import paper_2509_08309_amd as H

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("D,r", [(64, 1), (128, 2), (128, 8)])
def test_merge_segment_counts(D, r):
    chunk, counts = 16, [1, 2, 4, 5, 7, 8, 9, 31, 32, 33, 40, 63, 64, 65, 96, 97, 128, 129, 200, 0]
    lens = [16 * n - (n % 3) for n in counts]
    B, Hkv, cmax = len(counts), 2, max(counts)
    shape = H.make_shape(B, Hkv * r, Hkv, D, cmax)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(11)
    # [B, selected heads, chunks, r, D] and [B, selected heads, chunks, r]
    o_p = torch.randn((B, 2, cmax, r, D), generator=gen, device=DEV)
    lse = 3 * torch.randn((B, 2, cmax, r), generator=gen, device=DEV)
    for b, n in enumerate(counts):                      # what lies beyond a row's chunks is not read into it
        o_p[b, :, n:], lse[b, :, n:] = float("nan"), float("nan")
    sl = torch.tensor(lens, dtype=torch.int32, device=DEV)
    heads = [1, 0]
    out = torch.full((B, Hkv * r, D), 7.0, dtype=torch.float16, device=DEV)
    H.check(H.hetis_attn_merge(shape, o_p, lse, sl, torch.tensor(heads, dtype=torch.int32, device=DEV), 2, chunk,
                               cmax * 16, out), "merge")
    got = out.cpu().double().numpy().reshape(B, Hkv, r, D)
    o64, l64 = o_p.cpu().double().numpy(), lse.cpu().double().numpy()
    for b, n in enumerate(counts):
        for i, h in enumerate(heads):
            if n == 0:
                assert (got[b, h] == 0).all()
                continue
            w = np.exp(l64[b, i, :n] - l64[b, i, :n].max(axis=0))
            ref = (w[..., None] * o64[b, i, :n]).sum(axis=0) / w.sum(axis=0)[:, None]
            # half an fp16 ulp of the value, and n fp32 roundings (weights at 2^-21) of terms up to 5
            tol = np.abs(ref) * 2.0 ** -11 + 5 * (n + 4) * 2.0 ** -21 + 2.0 ** -25
            assert (np.abs(got[b, h] - ref) <= tol).all(), (n, h, np.abs(got[b, h] - ref).max())
