"""Tail sort and record fill at the edges of flows a thread, of windows of 256 records and of entries, against the CPU oracle: whole numbers, compared exactly."""
import numpy as np
import pytest
import torch

import oracle
import paper_2510_19262_amd as rs

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("M,N,B,C,kind", [
    (2, 4, 700, 4096, "tiny"),          # dozens of instances in a window, some of tails only, some empty
    (2, 2, 900, 4096, "tails"),         # no full chunk anywhere
    (40, 2, 30, 4096, "empty"),         # most instances without a record
    (2, 1, 1, 256, "long"),             # four flows, 60 000 records: entries far apart
    (3, 3, 2, 1000, "long"),            # nothing a power of two
    (16, 8, 1, 64, "dense"),            # a flow starts at every other record: several rounds of 64 starts in a window
    (33, 5, 3, 4096, "gaps"),           # hundreds of flows without a full chunk between long ones
    (8, 8, 3, 4096, "dense"),           # 512 flows: the most of two a thread of the tail sort
    (24, 8, 3, 100_000, "dense"),       # 1536, tails of 17 bits in three passes
    (64, 8, 1, 65536, "dense"),         # 4096: the most of four a thread
    (130, 8, 2, 65536, "dense"),        # 8320
    (4, 64, 2, 1000, "dense"),          # 16384: the most there can be
])
@pytest.mark.parametrize("shift", [0, 1])                            # record arrays on a 16-byte boundary and off it
def test_fill(M, N, B, C, kind, shift):
    G = M * N
    rng = np.random.default_rng(M * 100 + N)
    shape = (B, G, G)
    if kind == "tiny":
        D1n = np.where(rng.random(shape) < 0.6, 0, rng.integers(0, 3 * C, size=shape))
        D1n[::7] = 0
        D1n[3::7] %= C
    elif kind == "tails":
        D1n = rng.integers(0, C, size=shape)
    elif kind == "empty":
        D1n = np.where(rng.random((B, G, 1)) < 0.97, 0, rng.integers(0, 40 * C, size=shape))
    elif kind == "long":
        D1n = rng.integers(0, 60000 // max(1, G // 2) * C, size=shape)
    elif kind == "dense":
        D1n = rng.integers(0, 4 * C, size=shape)
    else:
        D1n = np.where(rng.random(shape) < 0.004, rng.integers(300 * C, 900 * C, size=shape), rng.integers(0, 2, size=shape) * (C - 1))
    D1n = D1n.astype(np.int64)
    off, w, flow, perm = oracle.chunk_sort_batch(D1n, M, N, C)
    n = int(off[-1])
    topo = rs.Topo(M, N, C)
    D1 = torch.from_numpy(D1n).to(DEV)
    for extra, want_perm in ((0, True), (1 << 21, True), (3, False)):    # no room to spare, and so much that there are entries
        cap = n + extra
        recs = [torch.full((cap + 9,), -7, dtype=torch.int32, device=DEV) for _ in range(3)]
        o = torch.empty(B * M + 1, dtype=torch.int64, device=DEV)
        arrays = [r[shift:shift + cap] for r in recs]
        rs.chunk_sort(D1, topo, capacity=cap, out=(o, arrays[0], arrays[1], arrays[2] if want_perm else None))
        assert np.array_equal(o.cpu().numpy(), off)
        for name, r, ref in zip(("w", "flow", "perm"), recs, (w, flow, perm)):
            h = r.cpu().numpy()
            if name == "perm" and not want_perm:
                assert (h == -7).all()
                continue
            assert np.array_equal(h[shift:shift + n].view(np.uint32), ref), (name, cap)
            assert (h[:shift] == -7).all() and (h[shift + n:] == -7).all(), name    # nothing outside the records


def test_fill_without_a_bound_on_capacity():
    # a capacity beyond any memory says that the arrays are large enough: the records are written in rounds of a smaller grid
    M, N, C = 4, 2, 64
    G = M * N
    gen = torch.Generator(device=DEV).manual_seed(5)
    D1 = torch.randint(0, 2 * 120_000_000 // (G * G) * C, (1, G, G), device=DEV, generator=gen)
    topo = rs.Topo(M, N, C)
    off, w, flow, perm = rs.chunk_sort(D1, topo)
    n = int(off[-1].item())
    assert n > (1 << 16) * 1024
    got = [torch.zeros(n, dtype=torch.int32, device=DEV) for _ in range(3)]
    o = torch.empty_like(off)
    rs.chunk_sort(D1, topo, capacity=1 << 62, out=(o, *got))
    assert torch.equal(o, off)
    for a, b in zip(got, (w, flow, perm)):
        assert torch.equal(a, b[:n])


@pytest.mark.parametrize("shift", [0, 1])
def test_fill_instances_around_a_window(shift):
    # one flow an instance, of as many full chunks as a window has, a few more or fewer, or hardly any, at every alignment
    M, N, B, C = 2, 1, 400, 4096
    rng = np.random.default_rng(3)
    q = rng.choice([0, 0, 1, 2, 3, 7, 252, 253, 254, 255, 256, 257, 258, 259, 260, 511, 512, 513, 5000], size=(B, 2))
    D1n = np.zeros((B, 2, 2), dtype=np.int64)
    D1n[:, [0, 1], [1, 0]] = q * C + rng.integers(0, 2, size=(B, 2)) * rng.integers(1, C, size=(B, 2))
    off, w, flow, perm = oracle.chunk_sort_batch(D1n, M, N, C)
    n = int(off[-1])
    D1 = torch.from_numpy(D1n).to(DEV)
    for cap in (n, n + (1 << 21)):                                       # without entries and with them
        recs = [torch.full((cap + 9,), -7, dtype=torch.int32, device=DEV) for _ in range(3)]
        o = torch.empty(B * M + 1, dtype=torch.int64, device=DEV)
        rs.chunk_sort(D1, rs.Topo(M, N, C), capacity=cap, out=(o, *[r[shift:shift + cap] for r in recs]))
        assert np.array_equal(o.cpu().numpy(), off)
        for name, r, ref in zip(("w", "flow", "perm"), recs, (w, flow, perm)):
            h = r.cpu().numpy()
            assert np.array_equal(h[shift:shift + n].view(np.uint32), ref), (name, cap)
            assert (h[:shift] == -7).all() and (h[shift + n:] == -7).all(), name


@pytest.mark.parametrize("M,N", [(2, 1), (8, 8)])                    # few flows, without room for counters, and many
@pytest.mark.parametrize("capacity", [0, 1 << 40])
@pytest.mark.parametrize("perm", [True, False])                      # half of the workgroups draw, or all
def test_fill_beyond_the_launch(M, N, capacity, perm):
    # more records than the launch has workgroups for: its last ones draw the rest by tickets, or go round.  Matrix by matrix there are fewer, and the records are the same
    B, C, G = 5, 4096, M * N
    per = 2 * 12_000_000 // (G * (G - N))                                # twice the mean number of chunks of a flow
    D1 = torch.randint(0, per * C, (B, G, G), device=DEV, generator=torch.Generator(device=DEV).manual_seed(M))
    if M == 2:
        D1[:, 0, 1] = 11_000_000 * C + 5
        D1[:, 1, 0] = torch.arange(B, device=DEV) * C + 77
    topo = rs.Topo(M, N, C)
    off = rs.chunk_count(D1, topo)
    n = int(off[-1].item())
    assert n > (1 << 15) * 1024 + 2_000_000
    out = (torch.empty_like(off), *[torch.full((n + 64,), -7, dtype=torch.int32, device=DEV) for _ in range(3)],
           torch.full((n + 64,), 99, dtype=torch.uint8, device=DEV), *[torch.empty((B, M, N), dtype=torch.int64, device=DEV) for _ in range(2)],
           torch.empty((B, 8), dtype=torch.int64, device=DEV))
    if not perm:
        out = (*out[:3], None, *out[4:])
    for _ in range(2):                                                   # the second time on counters that have been drawn on
        for t in out[1:5]:
            if t is not None:
                t.fill_(99)
        rs.schedule(D1, topo, capacity or n, out=out)
        assert torch.equal(out[0], off)
        for t in out[1:5]:
            assert t is None or (t[n:] == 99).all()
        for b in range(B):
            lo, hi = int(off[b * M].item()), int(off[(b + 1) * M].item())
            one = rs.schedule(D1[b:b + 1].contiguous(), topo, hi - lo)
            for name, a, r in zip(("w", "flow", "perm", "rail"), out[1:5], one[1:5]):
                assert a is None or torch.equal(a[lo:hi], r[:hi - lo]), (name, b)
            for a, r in zip(out[5:], one[5:]):
                assert torch.equal(a[b:b + 1], r)


@pytest.mark.parametrize("B", [8192, 8193, 16401])                   # the scan alone and with sums, of 2 nodes each
@pytest.mark.parametrize("large", [0, 9_000_000])                    # and with more records than the launch has workgroups for, beside its tickets
def test_offsets_of_many_instances(B, large):
    M, N, C, parts = 2, 1, 4096, 5
    rng = np.random.default_rng(B)
    q = rng.integers(0, 4, size=(B, 2)) * (rng.random((B, 2)) < 0.7)
    q[rng.choice(B, size=4, replace=False), 0] = 1000 + large
    D1n = np.zeros((B, 2, 2), dtype=np.int64)
    D1n[:, [0, 1], [1, 0]] = q * C + rng.integers(0, 2, size=(B, 2)) * rng.integers(1, C, size=(B, 2))
    D1 = torch.from_numpy(D1n).to(DEV)
    topo = rs.Topo(M, N, C)
    ref = np.concatenate([[0], np.cumsum((D1n[:, [0, 1], [1, 0]] + C - 1) // C)])
    assert np.array_equal(rs.chunk_count(D1, topo).cpu().numpy(), ref)
    n = int(ref[-1])
    for cap in (n, n + (1 << 21)):                                       # without entries and with them
        off, *recs = rs.chunk_sort(D1, topo, capacity=cap)
        assert np.array_equal(off.cpu().numpy(), ref)
        for p in range(parts):                                           # few enough instances for the scan alone
            b0, b1 = B * p // parts, B * (p + 1) // parts
            lo, hi = int(ref[b0 * M]), int(ref[b1 * M])
            _, *part = rs.chunk_sort(D1[b0:b1].contiguous(), topo, capacity=hi - lo)
            for name, a, r in zip(("w", "flow", "perm"), recs, part):
                assert torch.equal(a[lo:hi], r[:hi - lo]), (name, p, cap)


def test_fill_positions_above_31_bits():
    # one instance of more than 2^31 full chunks of one byte: entries are counted in 64 bits, positions go up to the last window
    topo = rs.Topo(1, 2, 1, include_intra_node=1)
    q = [(1 << 30) + 3, 5, (1 << 30) + 70_001, 1000]
    n = sum(q)
    assert n > 1 << 31
    D1 = torch.tensor(q, dtype=torch.int64, device=DEV).view(1, 2, 2)
    w = torch.zeros(n + 8, dtype=torch.int32, device=DEV)
    flow = torch.full((n + 8,), -7, dtype=torch.int32, device=DEV)
    off = torch.empty(2, dtype=torch.int64, device=DEV)
    rs.chunk_sort(D1, topo, capacity=n, out=(off, w, flow, None))
    assert off.tolist() == [0, n]
    assert (w[:n] == 1).all() and (w[n:] == 0).all() and (flow[n:] == -7).all()
    at = 0
    for f, c in enumerate(q):
        assert (flow[at:at + c] == f).all(), f
        at += c
