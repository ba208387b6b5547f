"""The fp32 attention kernel at the edges of its tiles, row groups and splits, against the oracle."""
from __future__ import annotations

import sys

import numpy as np
import pytest
import torch

import oracle
import paper_2608_24004_amd as av
import workload
from gpu_common import assert_attention_close, gpu_attention, to_host_f64
from helpers import random_paged

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# (label, (Hq, Hkv, D), contexts, drafts, window, KV blocks per split, sinks)
CASES = [
    ("one row", (1, 1, 128), [1, 15, 16, 300], [0, 0, 0, 0], 0, 0, False),
    ("one and two tiles", (32, 8, 128), [63, 40, 17, 900], [3, 4, 7, 8], 0, 3, True),
    ("three tiles, then a second row group", (16, 2, 128), [700, 129, 31], [5, 6, 13], 0, 0, False),
    ("window", (64, 8, 128), [2000, 130, 15], [2, 8, 4], 40, 2, True),
    ("four tiles, then a second row group", (64, 8, 64), [333, 512, 60], [7, 8, 0], 0, 5, False),
    ("all tile counts, D 64", (16, 2, 64), [90, 400, 1300, 35, 2], [1, 3, 5, 7, 1], 0, 0, True),
    ("more than 64 blocks per wavefront", (2, 1, 64), [4200, 30], [1, 0], 0, 300, False),
    ("more than 64 splits", (4, 1, 64), [1200, 1100], [2, 0], 0, 1, True),
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
@pytest.mark.parametrize("unmapped", [False, True], ids=["mapped", "unmapped"])
def test_f32_walk_edges(case, unmapped):
    label, (hq, hkv, d), contexts, drafts, window, split, with_sinks = case
    print("f32 walk", label, unmapped, file=sys.stderr, flush=True)
    p = random_paged(num_q_heads=hq, num_kv_heads=hkv, head_dim=d, dtype="f32", contexts=contexts, drafts=drafts,
                     window=window, seed=len(contexts) + d)
    bt = p.block_tables.copy()
    if unmapped:  # of several wavefronts, and a request's last block
        for i, s in enumerate(p.seq_lens):
            nb = (int(s) + 15) // 16
            bt[i, [b for b in (i % 4, nb // 2, nb - 1) if b < nb][: 1 + i % 3]] = -1 - i
    rng = np.random.default_rng(d + window)
    sinks = (rng.standard_normal(hq) * 2).astype(np.float32) if with_sinks else None
    args = p.oracle_args()
    args.update(block_tables=bt, sinks=sinks)
    ref = oracle.attention(**args)
    t = lambda a: torch.as_tensor(a, device=DEV)
    # the callers' tensors need only be aligned to a float
    odd = lambda x: torch.empty(x.numel() + 1, dtype=x.dtype, device=DEV)[1:].view(x.shape).copy_(x)
    q, kc, vc = odd(p.q), p.k_cache.to(DEV), p.v_cache.to(DEV)
    kw = dict(max_q_len=int(np.diff(p.q_start).max()), max_seq_len=int(p.seq_lens.max()))
    t_sinks = None if sinks is None else t(sinks)
    out = gpu_attention(q, kc, vc, t(bt), t(p.seq_lens), t(p.q_start), window=window, split=split, sinks=t_sinks, **kw)
    assert_attention_close(to_host_f64(out), ref, "f32", label)
    # the same through the fused append: the new tokens' K/V handed over, the cache without them
    new = [torch.empty((p.total_q, hkv, d), dtype=torch.float32) for _ in range(2)]
    stale_k, stale_v = p.k_cache.clone(), p.v_cache.clone()
    for i, s in enumerate(p.seq_lens):
        q0, n = int(p.q_start[i]), int(p.q_start[i + 1] - p.q_start[i])
        for dst, src in zip(new, (p.k_logical, p.v_logical)):
            dst[q0:q0 + n] = src[i][-n:].to(torch.float32)
        for pos in range(int(s) - n, int(s)):
            b = p.block_tables[i, pos // 16]
            stale_k[b, :, :, pos % 16] = 7.0
            stale_v[b, :, :, pos % 16] = -7.0
    kc2, vc2 = stale_k.to(DEV), stale_v.to(DEV)
    out2 = av.verify_attention_append(q, odd(new[0]), odd(new[1]), kc2, vc2, t(bt), t(p.seq_lens), t(p.q_start),
                                      sliding_window=window, kv_split_blocks=split, sinks=t_sinks, **kw)
    torch.cuda.synchronize()
    # bit for bit what the separate append and attention give
    assert torch.equal(out2, out)
    if not unmapped:
        assert np.array_equal(workload.host_storage(kc2), workload.host_storage(kc))
        assert np.array_equal(workload.host_storage(vc2), workload.host_storage(vc))


@pytest.mark.parametrize("hq,hkv,d,contexts,draft,window", [
    (1, 1, 64, [3434 + 900 * i for i in range(12)], 2, 128), (2, 2, 128, [229, 600, 900, 1220], 3, 0),
    (16, 4, 64, [1500, 700], 4, 0),
])
def test_f32_splits_lose_nothing(hq, hkv, d, contexts, draft, window):
    """Cutting a request into splits adds to its error against 64 bits only the
    merge's own sums, a few per cent beside the scores': no split's weight goes
    through a logarithm of the size of the scores (that added an eighth)."""
    p = random_paged(num_q_heads=hq, num_kv_heads=hkv, head_dim=d, dtype="f32", contexts=contexts,
                     drafts=[draft] * len(contexts), window=window, seed=hq + d)
    t = lambda a: torch.as_tensor(a, device=DEV)
    args = (p.q.to(DEV), p.k_cache.to(DEV), p.v_cache.to(DEV), t(p.block_tables), t(p.seq_lens), t(p.q_start))
    kw = dict(max_q_len=draft + 1, max_seq_len=int(p.seq_lens.max()), window=window)
    ref = oracle.attention(**p.oracle_args())
    err = {}
    for split in (0, 1, 100000):
        out = to_host_f64(gpu_attention(*args, split=split, **kw))
        err[split] = np.linalg.norm(out - ref) / np.linalg.norm(ref)
    print("f32 splits", hq, hkv, d, window, err, file=sys.stderr, flush=True)
    assert err[0] <= 1.05 * err[100000] and err[1] <= 1.05 * err[100000]
