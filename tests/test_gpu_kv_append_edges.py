"""verify_kv_append at the edges of its token rounds and alignments, bit for bit against a scatter in torch."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import paper_2608_24004_amd as av

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32], ids=["bf16", "f32"])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("odd", [False, True], ids=["aligned", "element-aligned"])
def test_kv_append_rounds(dtype, d, odd):
    rng = np.random.default_rng(d)
    hkv, x = 3, 16 // torch.empty(0, dtype=dtype).element_size()
    n = np.array([1, 2, 0, 31, 32, 33, 17, 70])      # tokens: one round, its edges, three rounds
    S = n + np.array([0, 15, 4, 1, 16, 30, -5, 7])    # and a request whose first tokens have no position
    nb = (np.maximum(S, 0) + 15) // 16
    tables = np.full((len(n), int(nb.max())), -1, dtype=np.int32)
    ids = rng.permutation(int(nb.sum()) + 3).astype(np.int32)
    tables[np.arange(tables.shape[1])[None, :] < nb[:, None]] = ids[:int(nb.sum())]
    tables[5, 1] = -7                                  # an unmapped block
    tables[7, 2] = int(nb.sum()) + 3                   # and one past the pool
    q_start = np.concatenate([[0], np.cumsum(n)])
    T, blocks = int(q_start[-1]), int(nb.sum()) + 3
    make = lambda *shape: torch.as_tensor(rng.standard_normal(shape), dtype=torch.float32).to(dtype).to(DEV)
    k_new, v_new = make(T, hkv, d), make(T, hkv, d)
    kc, vc = make(blocks, hkv, d // x, 16, x), make(blocks, hkv, d, 16)
    want_k, want_v = kc.clone(), vc.clone()
    for i in range(len(n)):
        for j in range(int(n[i])):
            p = int(S[i] - n[i]) + j
            b = int(tables[i, p // 16]) if p >= 0 else -1
            if 0 <= b < blocks:
                want_k[b, :, :, p % 16] = k_new[q_start[i] + j].view(hkv, d // x, x)
                want_v[b, :, :, p % 16] = v_new[q_start[i] + j]
    if odd:
        k_new, v_new = (torch.empty(t.numel() + 1, dtype=dtype, device=DEV)[1:].view(t.shape).copy_(t)
                        for t in (k_new, v_new))
    t32 = lambda a: torch.as_tensor(a, dtype=torch.int32, device=DEV)
    av.verify_kv_append(k_new, v_new, kc, vc, t32(tables), t32(S), t32(q_start))
    torch.cuda.synchronize()
    assert torch.equal(kc.view(torch.uint8), want_k.view(torch.uint8))
    assert torch.equal(vc.view(torch.uint8), want_v.view(torch.uint8))
