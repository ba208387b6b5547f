"""The bf16 walk at the edges of its dispatch, against the oracle.

Launches of short pairs give every (request, KV head, row group) pair to one
workgroup (the plan reports units_per_workgroup -1); others cut the walk into
ranges, and a few pairs cut into many slots are merged by thread groups that
share a row.  The walk itself goes in steps of two blocks, with single blocks
where a pair, a range or the mapped blocks end.
"""
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

# (label, (Hq, Hkv, D), contexts, drafts, window, sinks, expect whole pairs)
CASES = [
    ("16 blocks", (32, 8, 128), [251, 0, 15, 16, 17, 33, 240], [4, 0, 0, 3, 8, 4, 0], 0, False, True),
    ("17 blocks, few pairs", (8, 2, 128), [260, 31], [4, 0], 0, False, False),
    ("window of 9 to 10 blocks", (64, 8, 64), [4000, 130, 17, 900, 143], [5, 0, 16, 9, 8], 128, True, True),
    ("window, one row group too few", (16, 2, 64), [300, 90, 40], [31, 0, 2], 20, False, True),
    # twelve rows at most: one tile, whose pairs are cut beyond 28 blocks
    ("63 blocks, pairs on every CU", (32, 8, 128), [1000 - 31 * i for i in range(32)], [i % 3 for i in range(32)],
     0, True, False),
    ("63 blocks, two tiles, pairs on every CU", (32, 8, 128), [1000 - 31 * i for i in range(32)],
     [i % 6 for i in range(32)], 0, True, True),
    ("28 blocks, one tile, one long", (32, 8, 128), [445] + [3 * i for i in range(31)], [i % 3 for i in range(32)],
     0, True, True),
    ("69 blocks, more pairs than CUs", (64, 8, 64), [1100] + [13 * i + 1 for i in range(36)], [i % 3 for i in range(37)],
     0, True, True),
    ("64 blocks", (32, 8, 128), [1019, 500, 31, 1], [4, 8, 0, 2], 0, False, False),
    ("many slots per pair", (32, 8, 128), [2999, 16], [4, 0], 0, True, False),
    ("many slots per pair, D 64", (64, 8, 64), [3100], [8], 0, True, False),
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
@pytest.mark.parametrize("unmapped", [False, True], ids=["mapped", "unmapped"])
def test_walk_edges(case, unmapped):
    label, (hq, hkv, d), contexts, drafts, window, with_sinks, whole = case
    print("walk", label, unmapped, file=sys.stderr, flush=True)
    p = random_paged(num_q_heads=hq, num_kv_heads=hkv, head_dim=d, dtype="bf16", contexts=contexts, drafts=drafts,
                     window=window, seed=len(contexts) + d)
    bt = p.block_tables.copy()
    if unmapped:  # odd and even blocks of the steps, and a request's last block
        for i, s in enumerate(p.seq_lens):
            nb = (int(s) + 15) // 16
            bt[i, [b for b in (i % 4, nb // 2, nb - 1) if b < nb][: 1 + i % 3]] = -1 - i
    rng = np.random.default_rng(d + window)
    sinks = (rng.standard_normal(hq) * 2).astype(np.float32) if with_sinks else None
    args = p.oracle_args()
    args.update(block_tables=bt, sinks=sinks)
    ref = oracle.attention(**args)
    q, kc, vc = p.q.to(DEV), p.k_cache.to(DEV), p.v_cache.to(DEV)
    t = lambda a: torch.as_tensor(a, device=DEV)
    kw = dict(max_q_len=int(np.diff(p.q_start).max()), max_seq_len=int(p.seq_lens.max()))
    plan = av.attention_plan(q, kc, t(bt), sliding_window=window, **kw)
    assert all((c["units_per_workgroup"] == -1) == whole for c in plan["classes"])
    out = gpu_attention(q, kc, vc, t(bt), t(p.seq_lens), t(p.q_start), window=window,
                        sinks=None if sinks is None else t(sinks), **kw)
    assert_attention_close(to_host_f64(out), ref, "bf16", label)
    # the same through the fused append: the new tokens' K/V handed over, the cache without them
    new = [torch.empty((p.total_q, hkv, d), dtype=torch.bfloat16) for _ in range(2)]
    for i in range(len(contexts)):
        q0, n = int(p.q_start[i]), int(p.q_start[i + 1] - p.q_start[i])
        for dst, src in zip(new, (p.k_logical, p.v_logical)):
            dst[q0:q0 + n] = src[i][-n:].to(torch.bfloat16)
    stale_k, stale_v = p.k_cache.clone(), p.v_cache.clone()
    for i, s in enumerate(p.seq_lens):
        for pos in range(int(s) - int(p.q_start[i + 1] - p.q_start[i]), int(s)):
            b = p.block_tables[i, pos // 16]
            stale_k[b, :, :, pos % 16] = 7.0
            stale_v[b, :, :, pos % 16] = -7.0
    kc2, vc2 = stale_k.to(DEV), stale_v.to(DEV)
    out2 = av.verify_attention_append(q, new[0].to(DEV), new[1].to(DEV), kc2, vc2, t(bt), t(p.seq_lens), t(p.q_start),
                                      sliding_window=window, sinks=None if sinks is None else t(sinks), **kw)
    torch.cuda.synchronize()
    assert_attention_close(to_host_f64(out2), ref, "bf16", label + " append")
    if not unmapped:
        assert np.array_equal(workload.host_storage(kc2), workload.host_storage(kc))
        assert np.array_equal(workload.host_storage(vc2), workload.host_storage(vc))


@pytest.mark.parametrize("hq,hkv,d,window", [(8, 2, 64, 0), (32, 8, 128, 0), (16, 2, 64, 30)])
def test_walk_rows_past_max_q_len(hq, hkv, d, window):
    """More rows than max_q_len in a merged and in a whole-pair launch: the rows
    the plan reaches are computed (all of them: a tile beyond max_q_len too),
    the rest are NaN."""
    p = random_paged(num_q_heads=hq, num_kv_heads=hkv, head_dim=d, dtype="bf16", contexts=[900, 40, 2000],
                     drafts=[16, 9, 8], window=window, seed=hq)
    t = lambda a: torch.as_tensor(a, device=DEV)
    q, kc, vc = p.q.to(DEV), p.k_cache.to(DEV), p.v_cache.to(DEV)
    kw = dict(max_q_len=5, max_seq_len=int(p.seq_lens.max()))
    plan = av.attention_plan(q, kc, t(p.block_tables), sliding_window=window, **kw)
    reach = plan["row_groups"] * plan["rows_per_group"]
    out = to_host_f64(gpu_attention(q, kc, vc, t(p.block_tables), t(p.seq_lens), t(p.q_start), window=window, **kw))
    ref = oracle.attention(**p.oracle_args())
    G = hq // hkv
    row = np.concatenate([np.arange(n) for n in np.diff(p.q_start)])
    local = row[:, None] * G + np.arange(hq)[None, :] % G
    assert (local >= reach).any()
    assert_attention_close(out[local < reach], ref[local < reach], "bf16", "reached")
    assert np.isnan(out[local >= reach]).all()


@pytest.mark.parametrize("hq,hkv,d,contexts,drafts", [
    (32, 8, 128, [1500], [4]), (32, 8, 128, [500], [4]), (64, 8, 64, [3100], [8]), (8, 1, 128, [900, 333], [4, 16]),
])
def test_walk_of_few_pairs_rounds_twice(hq, hkv, d, contexts, drafts):
    """Few pairs, cut into ranges that do not fill the chip: only the weights and
    the output are rounded to bf16, the partial outputs are not.  A rounding to
    bf16 has a relative error of 2^-7 / sqrt(12) / m for a mantissa m, 1.6e-3 in the
    root mean square over [1, 2): 2.26e-3 for two of them, 2.76e-3 for three.  The
    line lies between."""
    p = random_paged(num_q_heads=hq, num_kv_heads=hkv, head_dim=d, dtype="bf16", contexts=contexts, drafts=drafts,
                     seed=hq + d)
    t = lambda a: torch.as_tensor(a, device=DEV)
    q, kc, vc = p.q.to(DEV), p.k_cache.to(DEV), p.v_cache.to(DEV)
    kw = dict(max_q_len=int(np.diff(p.q_start).max()), max_seq_len=int(p.seq_lens.max()))
    assert av.attention_plan(q, kc, t(p.block_tables), **kw)["units_per_workgroup"] == 0
    out = to_host_f64(gpu_attention(q, kc, vc, t(p.block_tables), t(p.seq_lens), t(p.q_start), **kw))
    ref = oracle.attention(**p.oracle_args())
    err = np.linalg.norm(out - ref) / np.linalg.norm(ref)
    print("two roundings", hq, hkv, d, contexts, "error %.3e" % err, file=sys.stderr, flush=True)
    assert err < 2.5e-3


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("hq,hkv,d,tokens,draft,window", [
    (32, 8, 128, 600, 4, 0), (8, 2, 64, 900, 8, 0), (8, 2, 128, 1500, 4, 512), (8, 1, 128, 2500, 16, 0),
])
def test_one_workspace_for_every_batch(dtype, hq, hkv, d, tokens, draft, window):
    """The workspace asked for the largest batch serves the smaller ones, whose
    pairs are cut where those of the largest are walked whole (bf16), or into more
    splits (fp32); nothing past its end is written."""
    B = 64
    p = random_paged(num_q_heads=hq, num_kv_heads=hkv, head_dim=d, dtype=dtype,
                     contexts=[tokens - 7 * (i % 5) for i in range(B)], drafts=[draft] * B, window=window, seed=d + hkv)
    t = lambda a: torch.as_tensor(a, device=DEV)
    q, kc, vc, bt = p.q.to(DEV), p.k_cache.to(DEV), p.v_cache.to(DEV), t(p.block_tables)
    kw = dict(max_q_len=draft + 1, max_seq_len=int(p.seq_lens.max()), sliding_window=window)
    n = av.attention_workspace_size(q, kc, bt, **kw)
    raw = torch.full((n + 4096,), 0xC3, dtype=torch.uint8, device=DEV)
    for b in (1, 2, 3, 5, 8, 13, 16, 20, 31, 40, 63, 64):
        print("one workspace", dtype, hkv, d, b, file=sys.stderr, flush=True)
        rows = b * (draft + 1)
        args = (q[:rows], kc, vc, bt[:b].contiguous(), t(p.seq_lens[:b]), t(p.q_start[:b + 1]))
        out = av.verify_attention(*args, workspace=raw[:n], **kw)
        assert torch.equal(out, av.verify_attention(*args, **kw))
        assert bool((raw[n:] == 0xC3).all())


@pytest.mark.parametrize("hq,hkv,d,contexts,drafts,bound,ranges", [
    (32, 8, 128, [40, 100, 5, 0, 63], [4, 0, 8, 2, 1], 16384, 500),  # fewer blocks than workgroups: ranges of one
    (64, 8, 64, [40, 100, 5, 0, 63], [4, 0, 8, 2, 1], 16384, 500),
    (8, 1, 128, [16000], [4], 16384, 80),                             # three rounds of the shared-row merge
    (8, 2, 64, [12000, 17], [8, 0], 16384, 80),
])
def test_walk_ranges(hq, hkv, d, contexts, drafts, bound, ranges):
    """A loose max_seq_len, whose plan has more workgroups than there are blocks,
    and long pairs cut into more slots than a round of the merge reads."""
    p = random_paged(num_q_heads=hq, num_kv_heads=hkv, head_dim=d, dtype="bf16", contexts=contexts, drafts=drafts,
                     seed=hq + d + len(contexts))
    t = lambda a: torch.as_tensor(a, device=DEV)
    q, kc, vc = p.q.to(DEV), p.k_cache.to(DEV), p.v_cache.to(DEV)
    kw = dict(max_q_len=int(np.diff(p.q_start).max()), max_seq_len=bound)
    print("walk ranges", hq, hkv, d, contexts, file=sys.stderr, flush=True)
    plan = av.attention_plan(q, kc, t(p.block_tables), **kw)
    assert plan["units_per_workgroup"] == 0 and plan["workgroups"] >= ranges
    if len(contexts) > 2:
        assert plan["workgroups"] > hkv * ((p.seq_lens + 15) // 16).sum()
    out = gpu_attention(q, kc, vc, t(p.block_tables), t(p.seq_lens), t(p.q_start), **kw)
    assert_attention_close(to_host_f64(out), oracle.attention(**p.oracle_args()), "bf16", "walk ranges")
