"""stream_receiver_stats keeps one softmax reference per row, set by the first tile in which a query sees
a key.  Scores hundreds of octaves above it overflow the row's sums: the row is then run again with
the true maxima.  Against the oracle, for each form of the row kernel, and for rows whose first tiles
hide every key (window, mask array)."""
import math

import numpy as np
import pytest
import torch

from oracle import receiver_stats as rs
from tests.test_gpu_receiver_stats import run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("bq,bk,mask,window", [(32, 32, "causal", 0), (64, 64, "causal", 0), (128, 32, "full", 0),
                                               (32, 128, "causal", 0), (128, 128, "sliding", 100)])
def test_scores_far_above_the_reference(dtype, bq, bk, mask, window):
    H, d = 3, 64
    T = 128 * 4 + 5
    print(f"[reference] {dtype} {bq}x{bk} {mask}", flush=True)
    g = torch.Generator().manual_seed(11)
    Q = torch.full((H, T, d), 4.0) + 0.25 * torch.randn((H, T, d), generator=g)
    K = torch.full((H, T, d), 6.0) + 0.25 * torch.randn((H, T, d), generator=g)
    K[:, :70] = 0.0            # the first tile's scores are 0; later ones 4 * 6 * 64 / 8 * log2(e) = 277 octaves
    K[:, 200:260] = -6.0       # ... and as far below
    Q, K = Q.to(dtype), K.to(dtype)
    scale = 1.0 / math.sqrt(d)
    got = run(Q, K, H, H, bq, scale, None, mask, window, block_k=bk)
    bm = got["block_mean"].astype(np.float64)
    assert np.isfinite(bm).all()
    t = np.arange(T)
    C = np.ones((T, T), bool) if mask == "full" else t[None, :] <= t[:, None]
    if mask == "sliding":
        C &= t[:, None] - t[None, :] < window
    for h in range(H):
        S = np.where(C, scale * (Q[h].double().numpy() @ K[h].double().numpy().T), -np.inf)
        P = np.exp(S - S.max(axis=1, keepdims=True))
        P /= P.sum(axis=1, keepdims=True)
        want, valid = rs.block_means(P, bq, mask, window, bk, None)
        # arguments of exp2 reach 600 octaves here: a few ulps of that in fp32 are 1e-4 of the value
        np.testing.assert_allclose(bm[h], want, rtol=1e-3, atol=1e-30)
        mean = want.sum(axis=0) / np.maximum(valid.sum(axis=0), 1)
        np.testing.assert_allclose(got["col_mean"][h], mean, rtol=1e-3, atol=1e-30)


def test_many_sequences_share_the_row_queue():
    """More row groups than workgroups in a round, sequences of 1 to 700 tokens, against each sequence alone."""
    from paper_2510_19875_amd import workloads as wl
    lens = tuple(1 + (i * 97) % 700 for i in range(40))
    w = wl.scaled(wl.config(5), lens, topk=1, heads=14, kv_heads=2, anchors_per_seq=0)
    Q, K, _, _ = wl.make_inputs(w, with_v=False)
    scale = 1.0 / math.sqrt(w.head_dim)
    got = run(Q, K, 14, 2, 64, scale, list(w.cu_seqlens))
    cu, b0 = w.cu_seqlens, 0
    for s, n in enumerate(lens):
        one = run(Q[:, cu[s]:cu[s + 1]].contiguous(), K[:, cu[s]:cu[s + 1]].contiguous(), 14, 2, 64, scale)
        nb = -(-n // 64)
        for key in ("col_mean", "col_kurt"):
            np.testing.assert_array_equal(got[key][:, b0:b0 + nb], one[key])
        np.testing.assert_array_equal(got["block_mean"][:, b0:b0 + nb, b0:b0 + nb], one["block_mean"])
        np.testing.assert_array_equal(got["head"][:, s], one["head"][:, 0])
        b0 += nb
