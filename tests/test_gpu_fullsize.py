"""Full-size workloads in the launch configuration bench.py times: sampled rows against the oracle
(rows are independent, so a sampled row is checked exactly) plus properties that hold at any size."""
import math

import numpy as np
import pytest
import torch

from oracle import stream_oracle as so
from paper_2510_19875_amd import binding, workloads as wl
from tests import parity

pytestmark = pytest.mark.gpu


def check_full(w, heads_sampled, n_rows, seed, check_sink=True, mask="causal", window=0):
    dev = torch.device("cuda:0")
    print(f"[full] {w.name}: generating inputs", flush=True)
    Q, K, V, meta = wl.make_inputs(w, device=dev)
    cu = w.cu_seqlens if w.batch > 1 else None
    topk = list(w.topk) if w.batch > 1 else w.topk[0]
    kmax = w.topk_max
    torch.cuda.reset_peak_memory_stats()
    base = torch.cuda.memory_allocated()
    print("[full] prune", flush=True)
    out = binding.stream_prune(Q, K, w.heads, w.kv_heads, w.block, topk, cu_seqlens=cu,
                               want_score=True, want_trace=True, mask=mask, window=window)
    scale = 1.0 / math.sqrt(w.head_dim)
    print("[full] attention", flush=True)
    att = binding.stream_sparse_attn(Q, K, V, w.heads, w.kv_heads, w.block, out["idx"], out["cnt"], scale,
                                     cu_seqlens=cu, want_lse=True, want_mass=True, mask=mask, window=window)
    torch.cuda.synchronize()
    extra = torch.cuda.max_memory_allocated() - base
    # O(T) memory: everything beyond the inputs is outputs + workspaces, linear in T (no T x T term)
    lin = (Q.numel() + 3 * K.numel()) * Q.element_size() + w.heads * w.T * 12 + \
        w.heads * w.total_blocks * kmax * (4 * 5 + 8 * out["levels"]) + (1 << 24)
    print(f"[full] extra device bytes {extra:,} (linear bound {lin:,})", flush=True)
    assert extra <= lin

    # ---- properties at full size
    bseq, bloc = so.block_table(w.cu_seqlens, w.block)
    qloc = torch.from_numpy(bloc).to(dev)
    kseq = torch.tensor([w.topk[s] for s in bseq], device=dev)
    cnt = out["cnt"]
    # valid key blocks of every row under the mask rule: rmin .. rmax
    nseq_blocks = torch.tensor([w.blocks_per_seq[s] for s in bseq], device=dev)
    rmax = nseq_blocks - 1 if mask == "full" else qloc
    rmin = torch.zeros_like(qloc)
    if mask == "sliding":
        lo = qloc * w.block - window + 1
        rmin = torch.where(lo > 0, torch.div(lo, w.block, rounding_mode="floor"), torch.zeros_like(lo))
    assert torch.equal(cnt, torch.minimum(kseq, rmax - rmin + 1).to(torch.int32)[None, :].expand_as(cnt))
    idx = out["idx"]
    slot = torch.arange(kmax, device=dev)[None, None, :]
    live = slot < cnt[:, :, None]
    assert bool(((idx >= rmin[None, :, None]) & (idx <= rmax[None, :, None]))[live].all()) and bool((idx[~live] == -1).all())
    assert bool((idx[:, :, 1:] > idx[:, :, :-1])[live[:, :, 1:]].all())
    if check_sink:
        assert bool((idx[:, :, 0] == 0).all())
    mass = att["mass"]
    assert bool((mass >= 0).all())
    np.testing.assert_allclose(mass.sum(dim=1).cpu().numpy(), float(w.T), rtol=2e-4)
    assert bool(torch.isfinite(att["O"].float()).all()) and bool(torch.isfinite(att["lse"]).all())

    # ---- sampled rows against the oracle (the rows of one head and sequence go to the oracle in
    #      one call: its row loop is the only thing it runs in parallel)
    rows = parity.sample_rows(w, n_rows, seed=seed, heads=heads_sampled)
    if not check_sink:
        # rows of the sampled heads that dropped block 0 (the planted sink) go to the oracle too
        lost = torch.nonzero((idx[heads_sampled, :, 0] != 0) & (cnt[heads_sampled] > 0))[:24].cpu().numpy()
        rows = sorted(set(rows) | {(heads_sampled[int(a)], int(b)) for a, b in lost})
        print(f"[full] {len(lost)} rows without block 0 added to the sample", flush=True)
    g = w.heads // w.kv_heads
    cuq = w.cu_seqlens
    idx_c, cnt_c = idx.cpu().numpy(), cnt.cpu().numpy()
    score_c, trace_c = out["score"].cpu().numpy(), out["trace"].cpu().numpy()
    tol = 2e-2 if w.dtype == "bf16" else 1e-4
    equal = ties = 0
    worst_o = worst_l = 0.0
    groups = {}
    for (h, gb) in rows:
        groups.setdefault((h, int(bseq[gb])), []).append(gb)
    for gi_, ((h, s), gbs) in enumerate(sorted(groups.items())):
        a, e = cuq[s], cuq[s + 1]
        Qh, Kh, Vh = (Q[h, a:e].float().cpu().numpy(), K[h // g, a:e].float().cpu().numpy(),
                      V[h // g, a:e].float().cpu().numpy())
        k = w.topk[s]
        ql = [int(bloc[gb]) for gb in gbs]
        r = so.prune_head(Qh, Kh, w.block, k, qblocks=ql, mask=mask, window=window)
        for i, gb in enumerate(gbs):
            q = ql[i]
            c = int(r["cnt"][i])
            assert c == int(cnt_c[h, gb])
            if np.array_equal(r["idx"][i], idx_c[h, gb, :k]):
                equal += 1
                np.testing.assert_allclose(score_c[h, gb, :c], r["score"][i, :c], rtol=1e-4)
            else:
                n_eff = max(1, math.ceil(math.log2(math.ceil(-(-(e - a) // w.block) / k))))
                ok, why = parity.certify_row(Qh, Kh, w.block, k, q, trace_c[:n_eff, h, gb, :k], mask=mask, window=window)
                assert ok, (h, gb, why)
                ties += 1
        # attention of those rows with the GPU's own lists (checked above) against Eq. (2) in fp64
        gi = np.ascontiguousarray(idx_c[h, gbs])
        gc = np.ascontiguousarray(cnt_c[h, gbs])
        ra = so.sparse_attn(Qh[None], Kh[None], Vh[None], 1, 1, w.block, gi, gc, scale,
                            rows=[(0, q) for q in ql], want_mass=False, mask=mask, window=window)
        O_h = att["O"][h, a:e].float().cpu().numpy()
        l_h = att["lse"][h, a:e].cpu().numpy()
        for q in ql:
            t0, t1 = q * w.block, min((q + 1) * w.block, e - a)
            worst_o = max(worst_o, float(np.abs(O_h[t0:t1] - ra["O"][0, t0:t1]).max()))
            worst_l = max(worst_l, float(np.abs(l_h[t0:t1] - ra["lse"][0, t0:t1]).max()))
        print(f"[full] group {gi_ + 1}/{len(groups)} (head {h}, sequence {s}): {len(gbs)} rows, "
              f"max|dO| so far {worst_o:.3e}", flush=True)
    print(f"[full] {w.name}: sampled rows={len(rows)} equal={equal} ties={ties} "
          f"max|dO|={worst_o:.3e} max|dlse|={worst_l:.3e}", flush=True)
    assert worst_o <= tol and worst_l <= 1e-3
    assert ties <= max(2, len(rows) // 20)
    return meta, att, (Q, K, V, idx_c, cnt_c)


def test_config2_real_shape_sampled():
    """T = 32,768, 32/8 heads, k = 16 at its own launch geometry (16,384 rows, 5 levels)."""
    # (k = 16: the sink's score is not among the 16 best of every row's first level, so block 0
    # is not always kept; the rows that dropped it are compared with the oracle)
    check_full(wl.config(2), heads_sampled=[1, 14, 22, 31], n_rows=520, seed=10, check_sink=False)


def test_config3_attention_and_prune_sampled():
    check_full(wl.config(3), heads_sampled=[2, 17, 30], n_rows=520, seed=11)


def test_config3_another_seeded_layer_sampled():
    """Config 3 is 32 independently seeded layers: one more of them (layer 17) against the oracle."""
    check_full(wl.config(3).with_layer(17), heads_sampled=[0, 11, 23], n_rows=320, seed=21, check_sink=False)


def test_config3_sliding_window_sampled():
    """The headline shape under a sliding window of 4096 tokens (65 valid key blocks per row,
    32 kept): the local layers of the Gemma 3 models the paper traces."""
    check_full(wl.config(3), heads_sampled=[4, 21], n_rows=256, seed=14, check_sink=False,
               mask="sliding", window=4096)


def test_config3_long_lists_sampled():
    """The headline tensors keeping 100 blocks per row: the kernels with the row's lists in LDS at scale."""
    w = wl.config(3)
    check_full(wl.scaled(w, w.seq_lens, topk=100, name=w.name + "_k100"), heads_sampled=[7, 25], n_rows=128, seed=15)


def test_config4_one_million_tokens_sampled():
    """T = 1,048,576, block 128, k = 64: O(T) memory and the four-wavefront row path at scale."""
    check_full(wl.config(4), heads_sampled=[5, 26], n_rows=512, seed=12)


def test_config5_ragged_reasoning_shape_sampled():
    w = wl.config(5)
    # (k_s is 1-5 here and the anchor keys outscore the sink, so block 0 is not always kept)
    meta, att, (Q, K, V, idx_c, cnt_c) = check_full(w, heads_sampled=[0, 9, 27], n_rows=560, seed=13, check_sink=False)
    # anchors (shared direction, every query has a component along it) collect far more mass
    mass = att["mass"].cpu().numpy()
    cu = w.cu_seqlens
    ratios = []
    for s in range(w.batch):
        a = [cu[s] + t for t in meta["anchors"][s]]
        ratios.append(np.median(mass[:, a]) / max(np.median(mass[:, cu[s]:cu[s + 1]]), 1e-9))
    print("[full] anchor/typical received-mass ratio per sequence:", np.round(ratios, 1), flush=True)
    assert np.median(ratios) > 5
    # per-key received mass, element by element: Eq. (2) over EVERY row of one (head, sequence)
    # pair in fp64 (with the kernel's own lists, checked above on the sampled rows), column sums
    # against the kernel's mass for that head over that sequence's keys
    g = w.heads // w.kv_heads
    scale = 1.0 / math.sqrt(w.head_dim)
    bseq, bloc = so.block_table(w.cu_seqlens, w.block)
    for (h, s) in ((9, int(np.argmax(w.seq_lens))), (22, int(np.argmin(w.seq_lens)))):
        a, e = cu[s], cu[s + 1]
        gbs = np.nonzero(bseq == s)[0]
        Qh, Kh, Vh = (Q[h, a:e].float().cpu().numpy(), K[h // g, a:e].float().cpu().numpy(),
                      V[h // g, a:e].float().cpu().numpy())
        ra = so.sparse_attn(Qh[None], Kh[None], Vh[None], 1, 1, w.block, np.ascontiguousarray(idx_c[h, gbs]),
                            np.ascontiguousarray(cnt_c[h, gbs]), scale, rows=[(0, int(bloc[gb])) for gb in gbs])
        m_ref, m_gpu = ra["mass"][0], mass[h, a:e]
        assert abs(m_ref.sum() - (e - a)) < 1e-6 * (e - a)
        # (fp32 atomics in no fixed order: 1e-3 relative, with a floor at 1e-3 of a uniform key's share)
        np.testing.assert_allclose(m_gpu, m_ref, rtol=1e-3, atol=1e-6)
        never = m_ref == 0
        assert (m_gpu[never] == 0).all()
        O_err = float(np.abs(att["O"][h, a:e].float().cpu().numpy() - ra["O"][0]).max())
        l_err = float(np.abs(att["lse"][h, a:e].cpu().numpy() - ra["lse"][0]).max())
        print(f"[full] config 5 head {h} sequence {s} ({e - a} tokens, k={w.topk[s]}): mass of every key "
              f"max rel err {float(np.max(np.abs(m_gpu - m_ref) / np.maximum(m_ref, 1e-3))):.2e}, "
              f"all {len(gbs)} rows: max|dO|={O_err:.3e} max|dlse|={l_err:.3e}", flush=True)
        assert O_err <= 2e-2 and l_err <= 1e-3


def test_attention_over_more_keys_than_one_launch_prepares():
    """64 kv heads of 4.2 M tokens: K and V are more than 2^24 groups of 32 keys.  The heads overlap in memory (16
    bytes apart), so that the inputs stay small; every query attends to its own block."""
    H, T, d, b = 64, (1 << 22) + 64, 64, 64
    N = T // b
    need = 2 * H * T * d * 2
    if torch.cuda.mem_get_info()[0] < need + (12 << 30):
        pytest.skip(f"{need >> 30} GiB of workspace do not fit beside what is in use")
    g = torch.Generator(device="cuda").manual_seed(6)
    flat = [torch.randn(T * d + 8 * H, generator=g, device="cuda").to(torch.bfloat16) for _ in range(4)]
    Q, K, V, O = (x.as_strided((H, T, d), (8, d, 1)) for x in flat)
    idx = torch.arange(N, dtype=torch.int32, device="cuda").expand(H, N)[..., None].contiguous()
    cnt = torch.ones((H, N), dtype=torch.int32, device="cuda")
    out = dict(O=O, lse=torch.empty((H, T), device="cuda"), mass=torch.full((H, T), 7.0, device="cuda"))
    print(f"[fullsize] preparation of {2 * H * T // 32} groups", flush=True)
    a = binding.stream_sparse_attn(Q, K, V, H, H, b, idx, cnt, 0.125, want_lse=True, want_mass=True, out=out)
    torch.cuda.synchronize()
    causal = torch.ones(b, b, dtype=torch.bool, device="cuda").tril()
    for h in (0, 31, 32, 63):
        for q in (0, N // 2, N - 1):
            rows = slice(q * b, q * b + b)
            S = (Q[h, rows].float() @ K[h, rows].float().T * 0.125).masked_fill(~causal, -math.inf)
            assert (a["lse"][h, rows] - S.logsumexp(1)).abs().max() <= 1e-3
            assert (a["mass"][h, rows] - S.softmax(1).sum(0)).abs().max() <= 1e-3
