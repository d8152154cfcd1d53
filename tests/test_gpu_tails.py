"""Tail sort at the edges of its workgroups, of counted and brought-together tails and of digits, against the CPU oracle: whole numbers, compared exactly."""
import numpy as np
import pytest
import torch

import oracle
import paper_2510_19262_amd as rs

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("M,N", [(65, 2), (8, 8), (57, 3), (16, 8), (257, 2), (20, 8), (144, 3), (24, 8), (97, 4), (32, 8), (33, 8), (48, 8), (49, 8), (64, 8), (65, 8),
                                 (128, 8), (17, 22), (16, 32)])       # N * N * M flows: both sides of every line
@pytest.mark.parametrize("C,span", [(4096, 1), (4096, 4095), (100_003, 100_002)])   # equal keys, two digits, three digits (17 bits)
def test_tails(M, N, C, span):
    G, NF = M * N, N * N * M
    rng = np.random.default_rng(NF + span)
    counts = [0, 1, 2, 63, 64, 65, 127, 128, 129, 130, 255, 256, 257, 511, 513, NF // 4, NF // 2 - 1, NF // 2, NF // 2 + 1, NF - 1, NF]
    B = -(-len(counts) // M)
    D1n = np.zeros((B, M, NF), dtype=np.int64)
    for i in range(B * M):
        nt = min(counts[i % len(counts)], NF)
        at = rng.choice(NF, size=nt, replace=False)
        D1n[i // M, i % M, at] = rng.integers(1, span + 1, size=nt)
    D1n += rng.integers(0, 3, size=D1n.shape) * (rng.random(D1n.shape) < 0.05) * C
    D1n = D1n.reshape(B, G, G)
    off, w, flow, perm = oracle.chunk_sort_batch(D1n, M, N, C, 1)
    n = int(off[-1])
    topo = rs.Topo(M, N, C, include_intra_node=1)
    o, *got = rs.chunk_sort(torch.from_numpy(D1n).to(DEV), topo, capacity=n + 5)
    assert np.array_equal(o.cpu().numpy(), off)
    for name, g, ref in zip(("w", "flow", "perm"), got, (w, flow, perm)):
        assert np.array_equal(g.cpu().numpy()[:n].view(np.uint32), ref), name
