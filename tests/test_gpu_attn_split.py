"""Few rows: the four wavefronts of a workgroup share a row of stream_sparse_attn; many rows: a row
each.  Both forms over the same heads, and head 0 against the oracle: lists shorter than the four
wavefronts, ragged tails, queries that see none of a wavefront's share, long lists, mask arrays."""
import math

import numpy as np
import pytest
import torch

from oracle import stream_oracle as so
from paper_2510_19875_amd import binding, workloads as wl

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
# O: half an ulp at |O| <= 4 (bf16) and the rounding of the probabilities; two forms differ by as much
# as either does from the oracle
TOL = {"bf16": 2e-2, "f32": 1e-4}


def documents(T):
    t = np.arange(T)
    doc = np.searchsorted(np.array([T // 5, T // 2, T // 2 + 40]), t, side="right")
    return (t[None, :] <= t[:, None]) & ((doc[:, None] == doc[None, :]) | (t[None, :] < 40))


def bits_of(C):
    T = C.shape[0]
    padded = np.zeros((T, -(-T // 32) * 32), dtype=np.uint8)
    padded[:, :T] = C
    return torch.from_numpy(np.packbits(padded, axis=1, bitorder="little").view(np.int32).copy()).to(DEV)


@pytest.mark.parametrize("T,block,k,dtype,d,mask", [
    (1013, 32, 1, "bf16", 128, "causal"),       # one sub-tile a row: three wavefronts have nothing
    (1013, 64, 3, "bf16", 128, "causal"),
    (2000, 128, 2, "bf16", 128, "sliding"),    # window edge: some queries see none of a share
    (1400, 64, 5, "bf16", 64, "documents"),
    (1999, 32, 7, "f32", 64, "causal"),
    (1100, 64, 3, "f32", 128, "documents"),
    (2500, 32, 65, "bf16", 128, "causal"),     # lists of more than 64 entries
    (2500, 32, 66, "bf16", 128, "documents"),
])
def test_shared_rows_match_whole_rows_and_the_oracle(T, block, k, dtype, d, mask):
    w = wl.scaled(wl.config(2), (T,), topk=k, heads=1, kv_heads=1, block=block, dtype=dtype, head_dim=d,
                  needles_per_kv_head=2)
    Q, K, V, _ = wl.make_inputs(w)
    C = documents(T) if mask == "documents" else None
    rule = dict(mask="sliding", window=150) if mask == "sliding" else {}
    Qf, Kf, Vf = Q.float().numpy(), K.float().numpy(), V.float().numpy()
    ref_kw = dict(C=C.astype(np.uint8)) if C is not None else rule
    lists = so.prune(Qf, Kf, 1, 1, block, k, **ref_kw)
    scale = 1.0 / math.sqrt(d)
    ref = so.sparse_attn(Qf, Kf, Vf, 1, 1, block, lists["idx"], lists["cnt"], scale, **ref_kw)
    gpu_kw = dict(mask_bits=bits_of(C)) if C is not None else rule

    def run(n):     # n equal heads: the number of rows decides which form runs
        print(f"[split] T={T} b={block} k={k} {dtype} {mask} heads={n}", flush=True)
        rep = lambda x: x.to(DEV).expand(n, -1, -1).contiguous()
        idx = torch.from_numpy(lists["idx"]).to(DEV).expand(n, -1, -1).contiguous()
        cnt = torch.from_numpy(lists["cnt"]).to(DEV).expand(n, -1).contiguous()
        a = binding.stream_sparse_attn(rep(Q), rep(K), rep(V), n, n, block, idx, cnt, scale, want_lse=True,
                                       want_mass=True, **gpu_kw)
        torch.cuda.synchronize()
        return [a[x].float().cpu().numpy() for x in ("O", "lse", "mass")]

    rows = -(-T // block) * (2 if block == 128 else 1)
    sub_tiles = k * max(1, block // 32)
    assert rows <= 60 * sub_tiles
    for O, lse, mass in (run(1), run(60 * sub_tiles // rows + 1)):
        assert np.abs(O - ref["O"]).max() <= TOL[dtype]
        np.testing.assert_array_equal(np.isneginf(lse), np.broadcast_to(np.isneginf(ref["lse"]), lse.shape))
        seen = ~np.isneginf(ref["lse"][0])
        assert np.abs(lse[:, seen] - ref["lse"][:, seen]).max() <= 1e-3
        assert (np.abs(mass - ref["mass"]) / np.maximum(ref["mass"], 1.0)).max() <= 1e-3


def steep(block, dtype, d, n_sub):
    """Heads whose scores lie near 0 but for two keys 110 to 140 octaves up, in 32-key sub-tiles of one
    wavefront's share or of two, ahead of or after sub-tiles without any."""
    octaves = (110.0, 118.0, 125.5, 126.5, 127.0, 127.625, 129.0, 140.0)
    places = ((1, 4), (4, 5), (4, 8), (5, 11))
    H, T = len(octaves) * len(places), 32 * n_sub - 27
    g = torch.Generator().manual_seed(3)
    Q, K, V = (torch.randn((H, T, d), generator=g) * s for s in (0.3, 0.3, 1.0))
    Q[:, :, :2] = 1.0
    K[:, :, :2] = 0.0
    for h in range(H):
        x, place = octaves[h % len(octaves)], places[h // len(octaves)]
        for i, sub in enumerate(place):
            key = 32 * sub + 3 + i
            K[h, key, 2:] = 0.0
            K[h, key, 0], K[h, key, 1] = int(x), x - int(x)
    ty = torch.bfloat16 if dtype == "bf16" else torch.float32
    return H, T, Q.to(ty), K.to(ty), V.to(ty)


@pytest.mark.parametrize("block,dtype,d,n_sub", [(32, "bf16", 128, 13), (64, "bf16", 128, 14), (128, "bf16", 64, 16),
                                                 (32, "f32", 64, 13), (64, "f32", 128, 14), (32, "bf16", 64, 66)])
def test_steep_scores(block, dtype, d, n_sub):
    """Sums up to 2^128 times their reference, on references up to 140 octaves apart: the weights of two keys
    that far above the rest are a half each, wherever they lie in a row and whichever form runs it."""
    H, T, Q, K, V = steep(block, dtype, d, n_sub)
    N = -(-T // block)
    idx = np.full((H, N, N), -1, np.int32)
    for q in range(N):
        idx[:, q, :q + 1] = np.arange(q + 1)
    cnt = np.broadcast_to(np.arange(1, N + 1, dtype=np.int32), (H, N)).copy()
    scale = math.log(2.0)
    ref = so.sparse_attn(Q.float().numpy(), K.float().numpy(), V.float().numpy(), H, H, block, idx, cnt, scale)
    rows, sub_tiles = H * N * (2 if block == 128 else 1), N * (block // 32)
    assert rows <= min(3000, 60 * sub_tiles)
    for n in (1, 60 * sub_tiles // rows + 1):
        print(f"[steep] b={block} {dtype} d={d} T={T} heads={H * n}", flush=True)
        rep = lambda x: x.to(DEV).repeat(n, 1, 1)
        a = binding.stream_sparse_attn(rep(Q), rep(K), rep(V), H * n, H * n, block, rep(torch.from_numpy(idx)),
                                       torch.from_numpy(cnt).to(DEV).repeat(n, 1), scale, want_lse=True, want_mass=True)
        torch.cuda.synchronize()
        for c in range(n):
            O, lse, mass = (a[x][c * H:(c + 1) * H].float().cpu().numpy() for x in ("O", "lse", "mass"))
            assert np.abs(O - ref["O"]).max() <= TOL[dtype]
            assert np.abs(lse - ref["lse"]).max() <= 1e-3
            assert (np.abs(mass - ref["mass"]) / np.maximum(ref["mass"], 1.0)).max() <= 1e-3


@pytest.mark.parametrize("T,block,k,slots,dtype,d,mask", [
    (1013, 32, 1, 64, "bf16", 128, "causal"),      # nearly empty lists: a row per wavefront after all
    (1013, 32, 32, 64, "bf16", 128, "causal"),     # full ones: shared
    (1990, 64, 2, 30, "bf16", 64, "sliding"),
    (1990, 64, 16, 30, "f32", 64, "causal"),
    (2000, 128, 1, 16, "bf16", 128, "documents"),
    (1111, 64, 17, 20, "f32", 128, "documents"),
    (2300, 32, 2, 66, "bf16", 128, "causal"),
    (2300, 32, 66, 70, "bf16", 64, "documents"),
])
def test_few_rows_go_by_their_lists(T, block, k, slots, dtype, d, mask):
    """Lists of k entries in `slots` slots, rows enough that the lists decide who shares."""
    w = wl.scaled(wl.config(2), (T,), topk=k, heads=1, kv_heads=1, block=block, dtype=dtype, head_dim=d,
                  needles_per_kv_head=2)
    Q, K, V, _ = wl.make_inputs(w)
    C = documents(T) if mask == "documents" else None
    rule = dict(mask="sliding", window=150) if mask == "sliding" else {}
    ref_kw = dict(C=C.astype(np.uint8)) if C is not None else rule
    Qf, Kf, Vf = Q.float().numpy(), K.float().numpy(), V.float().numpy()
    lists = so.prune(Qf, Kf, 1, 1, block, k, **ref_kw)
    scale = 1.0 / math.sqrt(d)
    ref = so.sparse_attn(Qf, Kf, Vf, 1, 1, block, lists["idx"], lists["cnt"], scale, **ref_kw)
    rows = -(-T // block) * (2 if block == 128 else 1)
    n = 800 // rows + 1
    assert 800 < n * rows <= min(3000, 60 * slots * max(1, block // 32))
    idx = np.full((1, lists["idx"].shape[1], slots), -1, np.int32)
    idx[:, :, :k] = lists["idx"]
    print(f"[split] T={T} b={block} k={k} of {slots} {dtype} {mask} heads={n}", flush=True)
    rep = lambda x: x.to(DEV).expand(n, -1, -1).contiguous()
    cnt = torch.from_numpy(lists["cnt"]).to(DEV).expand(n, -1).contiguous()
    a = binding.stream_sparse_attn(rep(Q), rep(K), rep(V), n, n, block, rep(torch.from_numpy(idx)), cnt, scale, want_lse=True,
                                   want_mass=True, **(dict(mask_bits=bits_of(C)) if C is not None else rule))
    torch.cuda.synchronize()
    O, lse, mass = (a[x].float().cpu().numpy() for x in ("O", "lse", "mass"))
    assert np.abs(O - ref["O"]).max() <= TOL[dtype]
    np.testing.assert_array_equal(np.isneginf(lse), np.broadcast_to(np.isneginf(ref["lse"]), lse.shape))
    seen = ~np.isneginf(ref["lse"][0])
    assert np.abs(lse[:, seen] - ref["lse"][:, seen]).max() <= 1e-3
    assert (np.abs(mass - ref["mass"]) / np.maximum(ref["mass"], 1.0)).max() <= 1e-3
