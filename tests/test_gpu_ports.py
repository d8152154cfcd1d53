"""Ports of chunks whose rails go round and round, with and without breaks in the round, against the CPU oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2510_19262_amd as rs

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("N", [1, 2, 3, 4, 8, 12, 16])
@pytest.mark.parametrize("P", [1, 2, 8, 128])
@pytest.mark.parametrize("kind", ["round", "breaks", "random end"])
def test_ports_of_rounds(N, P, kind):
    M, B = 3, 2
    rng = np.random.default_rng(N * 1000 + P)
    lens = rng.integers(1, 30_000, size=M * B)
    lens[1], lens[3] = 0, 1024
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    n = int(off[-1])
    rail = np.empty(n, dtype=np.uint8)
    for lo, hi in zip(off[:-1], off[1:]):
        r = np.arange(hi - lo) % N
        if kind == "breaks":                                         # the round starts anew, at another rail, at a few places
            for at in rng.integers(0, max(1, hi - lo), size=4):
                r[at:] = (np.arange(hi - lo - at) + rng.integers(0, N)) % N
        elif kind == "random end":
            r[len(r) * 3 // 4:] = rng.integers(0, N, size=len(r) - len(r) * 3 // 4)
        rail[lo:hi] = r
    topo = rs.Topo(M, N, 65536)
    got = rs.port_round_robin(torch.from_numpy(off).to(DEV), torch.from_numpy(rail).to(DEV), B, topo, P, capacity=n)
    assert np.array_equal(got.cpu().numpy()[:n], oracle.port_round_robin(off, rail, B, M, N, P))
