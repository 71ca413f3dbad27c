"""stream_receiver_stats keeps one softmax reference per row, set by the first tile in which a query sees
a key.  Scores hundreds of octaves above it overflow the row's sums: the row is then run again with
the true maxima.  Against the oracle, for each form of the row kernel, and for rows whose first tiles
hide every key (window, mask array)."""
import ctypes
import math

import numpy as np
import pytest
import torch

from oracle import receiver_stats as rs
from paper_2510_19875_amd import binding
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


def packed_copies(H, Hkv, T, d, b, bk, esize, array=False):
    """Bytes of packed copies of Q and K, 4 bytes per padded token and head, and a mask array's summaries."""
    pad, up = -(-T // max(b, bk)) * max(b, bk), lambda x: -(-x // 256) * 256
    n = up(H * pad * d * esize) + up(Hkv * pad * d * esize) + up(H * pad * 4)
    if array:
        n += 2 * up(pad // b * (-(-(pad // bk) // 32)) * 4) + up(H * (pad // bk) * 4)
    return n


@pytest.mark.parametrize("H,Hkv,T,d,b,bk,dtype,mask,steep", [
    (1, 1, 9001, 128, 64, 64, torch.bfloat16, "causal", False),
    (3, 1, 5003, 64, 32, 32, torch.bfloat16, "causal", True),
    (2, 2, 4100, 64, 128, 32, torch.float32, "sliding", False),
    (2, 1, 4100, 64, 32, 128, torch.bfloat16, "full", True),
    (2, 2, 3900, 64, 128, 128, torch.bfloat16, "sliding", True),
    (1, 1, 3001, 64, 64, 32, torch.bfloat16, "array", False),
    (1, 1, 40003, 64, 32, 32, torch.bfloat16, "causal", False),      # the span sums come in chunks
])
def test_a_workspace_without_scratch_rows(H, Hkv, T, d, b, bk, dtype, mask, steep):
    """Packed copies of Q and K are room enough, nothing beyond is written, and the results are those of the
    workspace that the query asks for."""
    print(f"[budget] H={H}/{Hkv} T={T} d={d} {b}x{bk} {dtype} {mask} steep={steep}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(4)
    Q, K = (torch.randn((n, T, d), generator=g, device="cuda") for n in (H, Hkv))
    if steep:
        Q[..., 0], K[..., 0] = 12.0, 0.0
        K[:, 300:, 0] = 12.0 * d ** 0.5                              # 200 octaves above the first tiles
    Q, K = Q.to(dtype), K.to(dtype)
    kw = dict(mask=mask, window=3000 if mask == "sliding" else 0)
    if mask == "array":
        t = torch.arange(T)
        from tests.test_gpu_mask_array import pack_bits
        kw["mask_bits"] = pack_bits(((t[None, :] <= t[:, None]) & (t[None, :] // 900 == t[:, None] // 900)).numpy())
    need = packed_copies(H, Hkv, T, d, b, bk, dtype.itemsize, mask == "array")
    room = torch.full((need + 65536,), 0x5A, dtype=torch.uint8, device="cuda")
    args = (Q, K, H, Hkv, b, 1.0 / math.sqrt(d))
    shape, _ = binding.make_shape(H, Hkv, d, b, binding._dtype_code(Q), T, None, Q=Q, K=K, block_k=bk, **kw)
    assert need < binding.load().stream_receiver_stats_workspace_bytes(ctypes.byref(shape))
    small = binding.stream_receiver_stats(*args, want_block_mean=True, block_k=bk, workspace=room[:need], **kw)
    large = binding.stream_receiver_stats(*args, want_block_mean=True, block_k=bk, **kw)
    torch.cuda.synchronize()
    assert bool((room[need:] == 0x5A).all())
    # sums of 64 probabilities per query tile in another order, their arguments a few ulps apart
    for key in ("block_mean", "col_mean"):
        torch.testing.assert_close(small[key], large[key], rtol=2e-4 if steep else 2e-5, atol=1e-30)
    for key in ("col_kurt", "head"):
        torch.testing.assert_close(small[key], large[key], rtol=1e-2, atol=1e-2)


@pytest.mark.parametrize("b,dtype", [(64, torch.bfloat16), (32, torch.bfloat16), (64, torch.float32)])
def test_error_against_64_bits(b, dtype):
    """Block means are averages over b x b probabilities with an error of a few 1e-8 each from the scores and
    exponentials; what the sums over a row and over a span add must stay below that.  The kurtosis of a column
    amplifies the errors of its largest entries by about four."""
    H, T, d = 4, 12288, 128
    print(f"[error] b={b} {dtype}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(8)
    Q, K = (torch.randn((H, T, d), generator=g, device="cuda") for _ in range(2))
    K[:, 0] *= 4.0
    Q, K = Q.to(dtype), K.to(dtype)
    got = binding.stream_receiver_stats(Q, K, H, H, b, 1.0 / math.sqrt(d), want_block_mean=True)
    N = T // b
    t = torch.arange(T, device="cuda")
    hidden = t[None, :] > t[:, None]
    visible = torch.ones(N, N, dtype=torch.bool, device="cuda").tril()
    n = visible.sum(0)
    for h in range(H):
        P = torch.softmax((Q[h].double() @ K[h].double().T / math.sqrt(d)).masked_fill_(hidden, -math.inf), 1)
        M = P.view(N, b, N, b).mean((1, 3))
        y = torch.where(visible, M - M.sum(0) / n, 0.0)
        kurt = torch.where(n >= 4, (y ** 4).sum(0) / n / ((y ** 2).sum(0) / n).clamp(min=1e-300) ** 2 - 3.0, 0.0)
        err = lambda a, w: float((a.double() - w).norm() / w.norm())
        e = err(got["block_mean"][h], M), err(got["col_kurt"][h], kurt)
        print(f"[error] head {h} {e[0]:.2e} {e[1]:.2e}", flush=True)
        assert e[0] <= 9e-8 and e[1] <= 2.8e-7
