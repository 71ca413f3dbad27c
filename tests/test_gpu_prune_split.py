"""Few rows: the four wavefronts of a workgroup share a row of stream_prune / stream_prune_multi /
stream_prune_variable; many rows: a row each.  Copies of one head decide which form runs; both must give
the same lists, scores, traces and counts of scored blocks bit for bit, and the oracle's lists."""
import numpy as np
import pytest
import torch

from oracle import stream_oracle as so
from paper_2510_19875_amd import binding, workloads as wl
from tests.test_gpu_attn_split import bits_of, documents

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

CASES = [
    (1013, 32, 16, "bf16", 128, "causal"),
    (70, 32, 3, "bf16", 128, "causal"),            # a level of fewer blocks than wavefronts
    (1999, 64, 5, "bf16", 128, "causal"),          # short lists: sub-tiles of a block
    (2000, 64, 9, "bf16", 64, "sliding"),
    (1500, 32, 6, "f32", 64, "causal"),
    (1111, 64, 4, "f32", 128, "causal"),
    (1400, 64, 5, "bf16", 128, "documents"),
    (2300, 32, 66, "bf16", 128, "causal"),         # lists in LDS
    (2300, 32, 70, "bf16", 128, "documents"),
    (4400, 64, 67, "bf16", 128, "sliding"),
]


def setup(T, block, k, dtype, d, mask):
    w = wl.scaled(wl.config(2), (T,), topk=k, heads=1, kv_heads=1, block=block, dtype=dtype, head_dim=d,
                  needles_per_kv_head=2)
    Q, K, _, _ = wl.make_inputs(w, with_v=False)
    C = documents(T) if mask == "documents" else None
    rule = dict(mask="sliding", window=500) if mask == "sliding" else {}
    gpu = dict(mask_bits=bits_of(C)) if C is not None else rule
    ref = dict(C=C.astype(np.uint8)) if C is not None else rule
    rows = -(-T // block)
    if k > 64:
        limit = 3000 if block == 32 else 1500
    else:
        limit = (80 if block == 32 else 64) * k
    assert rows <= limit
    return Q, K, gpu, ref, limit // rows + 1


@pytest.mark.parametrize("T,block,k,dtype,d,mask", CASES)
def test_shared_rows_equal_whole_rows_and_the_oracle(T, block, k, dtype, d, mask):
    Q, K, gpu, ref_kw, many = setup(T, block, k, dtype, d, mask)
    ref = so.prune(Q.float().numpy(), K.float().numpy(), 1, 1, block, k, **ref_kw)
    got = []
    for n in (1, many):
        print(f"[split] T={T} b={block} k={k} {dtype} {mask} heads={n}", flush=True)
        r = binding.stream_prune(Q.to(DEV).expand(n, -1, -1).contiguous(), K.to(DEV).expand(n, -1, -1).contiguous(), n, n,
                                 block, k, want_score=True, want_trace=True, want_tiles=True, **gpu)
        torch.cuda.synchronize()
        assert int(r["tiles"].item()) == n * int(ref["evals"][1])
        got.append(r)
    one, all_ = got
    for h in (0, many - 1):
        for x in ("idx", "cnt", "score"):
            assert torch.equal(one[x][0], all_[x][h])
        assert torch.equal(one["trace"][:, 0], all_["trace"][:, h])
    np.testing.assert_array_equal(one["cnt"].cpu().numpy(), ref["cnt"])
    np.testing.assert_array_equal(one["idx"].cpu().numpy(), ref["idx"])


@pytest.mark.parametrize("T,block,ks,mask", [(1500, 32, (16, 8, 3, 1), "causal"), (2000, 64, (2, 7, 5), "documents"),
                                             (1700, 64, (12, 1), "sliding")])
def test_sweep_and_variable_k(T, block, ks, mask):
    Q, K, gpu, _, _ = setup(T, block, max(ks), "bf16", 128, mask)
    rows = -(-T // block)
    multi = []
    for n in (1, 40 * max(ks) // rows + 2):
        Qn, Kn = Q.to(DEV).expand(n, -1, -1).contiguous(), K.to(DEV).expand(n, -1, -1).contiguous()
        multi.append(binding.stream_prune_multi(Qn, Kn, n, n, block, list(ks), want_score=True, want_tiles=True, **gpu))
        var = binding.stream_prune_variable(Qn, Kn, n, n, block, 1, 6, 1, max(ks), want_score=True, **gpu)
        multi[-1]["var"] = var
    torch.cuda.synchronize()
    one, all_ = multi
    n = all_["idx"].shape[0]
    assert int(all_["tiles"].item()) == n * int(one["tiles"].item())
    for x in ("idx", "cnt", "score"):
        assert torch.equal(one[x][0], all_[x][n - 1])
        assert torch.equal(one["var"][x][0], all_["var"][x][n - 1])
    for i, k in enumerate(ks):
        single = binding.stream_prune(Q.to(DEV), K.to(DEV), 1, 1, block, k, want_score=True, **gpu)
        assert torch.equal(one["idx"][0, i, :, :k], single["idx"][0])
        assert torch.equal(one["score"][0, i, :, :k], single["score"][0])


@pytest.mark.parametrize("block,T", [(32, 32 * 1100 - 9), (64, 64 * 2100 - 30)])
def test_sweep_over_more_blocks_than_the_score_cache_holds(block, T):
    """Blocks of one level that fall on the same entry of the row's score cache (1024 entries)."""
    ks = (64, 32, 7, 1)
    g = torch.Generator().manual_seed(9)
    Q, K = (torch.randn((1, T, 64), generator=g).to(torch.bfloat16).to(DEV) for _ in range(2))
    assert 1024 < -(-T // block) <= (20 if block == 32 else 40) * max(ks)
    print(f"[split] sweep T={T} b={block}", flush=True)
    multi = binding.stream_prune_multi(Q, K, 1, 1, block, list(ks), want_score=True)
    for i, k in enumerate(ks):
        one = binding.stream_prune(Q, K, 1, 1, block, k, want_score=True)
        torch.cuda.synchronize()
        assert torch.equal(multi["cnt"][0, i], one["cnt"][0])
        assert torch.equal(multi["idx"][0, i, :, :k], one["idx"][0])
        assert torch.equal(multi["score"][0, i, :, :k], one["score"][0])
