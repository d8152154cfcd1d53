"""Stages 3-5 at the edges of the per-instance kernels (threads per instance, tails counted or sorted, chains by runs, one workgroup per
instance or separate kernels), against the CPU oracle: whole numbers, compared exactly."""
import numpy as np
import pytest
import torch

import oracle
import paper_2510_19262_amd as rs

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _matrix(kind, B, G, C, rng):
    if kind == "payload":                            # few tail values, long runs of them, ties a full weight apart
        m = rng.poisson(3.0, size=(B, G, G)) * (C * 7 // 64)
    elif kind == "tokens":                           # most flows shorter than a chunk, many of none
        m = rng.poisson(0.7, size=(B, G, G)) * (C // 9 + 1)
    elif kind == "any":                              # every tail different
        m = rng.integers(0, 5 * C, size=(B, G, G))
    elif kind == "sparse":                           # long stretches of flows without full chunks between long flows
        m = np.where(rng.random((B, G, G)) < 0.01, rng.integers(20 * C, 90 * C, size=(B, G, G)), rng.integers(0, 3, size=(B, G, G)))
    else:                                            # "two": runs of two weights, the lighter far below the spread the heavier leaves
        m = np.where(rng.random((B, G, G)) < 0.5, C - 1, 3)
    return m.astype(np.int64)


@pytest.mark.parametrize("kind", ["payload", "tokens", "any", "sparse", "two"])
@pytest.mark.parametrize("M,N,B,C", [(4, 4, 1, 65536),            # 64 flows
                                     (3, 9, 2, 100_000),          # 243, nothing a power of two
                                     (4, 8, 2, 65536),            # 256
                                     (5, 8, 3, 4096),             # 320
                                     (16, 8, 2, 131072),          # 1024
                                     (17, 8, 1, 131072),          # 1088: 1024 threads
                                     (8, 16, 2, 65536),           # 2048, 16 rails
                                     (2, 32, 3, 65536),           # 2048, the list spans the wavefront
                                     (64, 8, 1, 131072),          # 4096: the largest in one workgroup
                                     (65, 8, 1, 131072),          # 4160: separate kernels
                                     (28, 12, 1, 262144),         # 4032, 12 rails
                                     (3, 8, 180, 65536),          # 540 instances of 192 flows: 256 threads up to 16 chunks a flow
                                     (2, 8, 390, 65536),          # 780 of 128
                                     (12, 12, 22, 65536),         # 264 of 1728: 512 threads
                                     (4, 2, 300, 4096),           # 1200 instances
                                     (16, 8, 66, 65536)])         # 1056 instances of 1024 flows
def test_instances(M, N, B, C, kind):
    G = M * N
    rng = np.random.default_rng(M * 1000 + N * 10 + B)
    D1n = _matrix(kind, B, G, C, rng)
    topo = rs.Topo(M, N, C)
    off, w, flow, perm = oracle.chunk_sort_batch(D1n, M, N, C)
    rail, S = oracle.lpt_batch(off, w, B, M, N)
    _, R, stats = oracle.eval_batch(off, w, flow, rail, B, M, N)
    n = int(off[-1])
    want = dict(off=off, w=w, flow=flow, perm=perm, rail=rail, S=S, R=R, stats=stats)
    D1 = torch.from_numpy(D1n).to(DEV)
    u32 = lambda t: t.cpu().numpy().view(np.uint32)[:n]

    def check(got, what):
        o, gw, gf, gp, gr, gS, gR, gst = got
        have = dict(off=o.cpu().numpy(), w=u32(gw), flow=u32(gf), perm=u32(gp), rail=gr.cpu().numpy()[:n], S=gS.cpu().numpy(),
                    R=gR.cpu().numpy(), stats=gst.cpu().numpy())
        for key, value in want.items():
            assert np.array_equal(have[key], value), f"{what} {key}"

    check(rs.schedule(D1, topo, n), "one call")
    o, gw, gf, gp = rs.chunk_sort(D1, topo)
    gr, gS = rs.lpt_spray(o, gw, B, topo)
    check((o, gw, gf, gp, gr, gS, *rs.eval(o, gw, gf, gr, gS, B, topo)), "three calls")
    # too little room by one record: the loads say so and no record is touched
    if n:
        out = rs.schedule(D1, topo, n - 1)
        assert (out[5].cpu().numpy() == -1).all() and (out[6].cpu().numpy() == -1).all() and (out[7].cpu().numpy() == -1).all()
        assert np.array_equal(out[0].cpu().numpy(), off)


@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("M,N,full", [(4, 4, [32768, 1, 0, 5]),                      # as many as a workgroup writes itself
                                      (4, 4, [33023, 32769, 33025, 40000]),          # around the boundary of the record arrays behind them
                                      (2, 5, [36864 + 32768, 50_001]),               # one tile and a ragged one, 5 rails
                                      (16, 16, [100_000] + [3] * 14 + [36_900]),     # 4096 flows
                                      (70, 2, [70] * 35 + [300_000] + [70] * 33 + [33_100])])   # the long ones among more than 64 instances
def test_long_instances_share_their_records(M, N, full, shift):
    # instances longer than the mean: further workgroups write part of their records
    G, C, B = M * N, 4096, 2
    rng = np.random.default_rng(M + N)
    D1n = rng.integers(0, C, size=(B, G, G)) * (rng.random((B, G, G)) < 0.5)          # tails
    for b in range(B):
        for k in range(M):                                                             # full chunks of node k over its flows to other nodes
            cols = np.r_[0:k * N, k * N + N:G]
            share = rng.multinomial(full[(k + b) % M], np.full(N * cols.size, 1.0 / (N * cols.size)))
            share[rng.random(share.size) < 0.3] = 0
            share[0] += full[(k + b) % M] - share.sum()
            D1n[b, k * N:k * N + N, cols] += (share.reshape(N, cols.size) * C).T
    D1n = D1n.astype(np.int64)
    topo = rs.Topo(M, N, C)
    off, w, flow, perm = oracle.chunk_sort_batch(D1n, M, N, C)
    rail, S = oracle.lpt_batch(off, w, B, M, N)
    _, R, stats = oracle.eval_batch(off, w, flow, rail, B, M, N)
    n = int(off[-1])
    D1 = torch.from_numpy(D1n).to(DEV)
    arrays = [torch.full((n + 8,), 77, dtype=dt, device=DEV) for dt in (torch.int32, torch.int32, torch.int32, torch.uint8)]
    lead = 4 - shift                                                                   # 1: off the 16-byte boundary, scalar stores
    gw, gf, gp, gr = (t[lead:lead + n] for t in arrays)
    out = (torch.empty(B * M + 1, dtype=torch.int64, device=DEV), gw, gf, gp, gr, torch.empty((B, M, N), dtype=torch.int64, device=DEV),
           torch.empty((B, M, N), dtype=torch.int64, device=DEV), torch.empty((B, 8), dtype=torch.int64, device=DEV))
    rs.schedule(D1, topo, n, out=out)
    u32 = lambda t: t.cpu().numpy().view(np.uint32)
    for name, got, want in (("off", out[0].cpu().numpy(), off), ("w", u32(gw), w), ("flow", u32(gf), flow), ("perm", u32(gp), perm),
                            ("rail", gr.cpu().numpy(), rail), ("S", out[5].cpu().numpy(), S), ("R", out[6].cpu().numpy(), R),
                            ("stats", out[7].cpu().numpy(), stats)):
        assert np.array_equal(got, want), name
    for t in arrays:
        assert (t[:lead] == 77).all() and (t[lead + n:] == 77).all()
    short = rs.schedule(D1, topo, n - 1)                                               # too little room: nobody writes records
    assert (short[5].cpu().numpy() == -1).all()
