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
