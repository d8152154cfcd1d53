"""What a call may cost beside another of the same work: ratios with wide margins, for costs that once were ten times as high."""
import statistics

import pytest
import torch

import paper_2510_19262_amd as rs

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _us(*calls):
    """Medians of 9 times of each call, taken in turn."""
    times = [[] for _ in calls]
    for r in range(11):
        for call, t in zip(calls, times):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(4):
                call()
            b.record()
            b.synchronize()
            if r >= 2:
                t.append(a.elapsed_time(b) * 250)
    return [statistics.median(t) for t in times]


def _matrices(M, N, B, C, mean, zero=0.0):
    gen = torch.Generator(device=DEV).manual_seed(M * B)
    shape = (B, M * N, M * N)
    D1 = (torch.rand(shape, device=DEV, generator=gen) * 2 * mean * C).to(torch.int64)
    return torch.where(torch.rand(shape, device=DEV, generator=gen) < zero, torch.zeros_like(D1), D1)


def _sort(D1, topo, n, capacity):
    out = (torch.empty(D1.shape[0] * topo.nodes + 1, dtype=torch.int64, device=DEV), *[torch.empty(n + 1, dtype=torch.int32, device=DEV) for _ in range(3)])
    ws = torch.empty(rs.chunk_sort_workspace_bytes(D1.shape[0], topo), dtype=torch.uint8, device=DEV)
    return lambda: rs.chunk_sort(D1, topo, capacity=capacity, out=out, ws=ws)


@pytest.mark.parametrize("M,N,B,mean", [(4, 4, 1, 20), (8, 8, 16, 150)])
@pytest.mark.parametrize("capacity", [400_000_000, 4_200_000_000, 1 << 62])
def test_room_that_is_not_used_costs_little(M, N, B, mean, capacity):
    topo = rs.Topo(M, N, 65536)
    D1 = _matrices(M, N, B, topo.chunk_bytes, mean)
    n = rs.chunk_total(D1, topo)
    tight, roomy = _us(_sort(D1, topo, n, n), _sort(D1, topo, n, capacity))
    assert roomy < 1.5 * tight + 20, (tight, roomy)                      # 20 / 27 and 33 / 40 us; 880 us when 4.2 G records had a workgroup a tile


@pytest.mark.parametrize("M,N,B,mean,zero", [(2, 1, 8000, 2, 0.95), (4, 4, 256, 2, 0.95), (3, 8, 1335, 2, 0.99), (11, 8, 87, 2, 0.99)])
def test_instances_of_few_records_cost_no_more_than_of_many(M, N, B, mean, zero):
    topo = rs.Topo(M, N, 65536)
    sparse, dense = _matrices(M, N, B, topo.chunk_bytes, mean, zero), _matrices(M, N, B, topo.chunk_bytes, 20)
    counts = [rs.chunk_total(D, topo) for D in (sparse, dense)]
    few, many = _us(*[_sort(D, topo, n, n) for D, n in zip((sparse, dense), counts)])
    assert few < 1.4 * many + 15, (few, many)                            # 2.5 to 15 times when a wavefront went from instance to instance


@pytest.mark.parametrize("M,N,B", [(130, 8, 4), (64, 8, 20), (30, 6, 130), (16, 8, 250)])
def test_few_tails_cost_less_than_many(M, N, B):
    topo = rs.Topo(M, N, 65536)
    gen = torch.Generator(device=DEV).manual_seed(M)
    many = torch.randint(1, topo.chunk_bytes, (B, M * N, M * N), device=DEV, generator=gen)
    few = torch.where(torch.rand(many.shape, device=DEV, generator=gen) < 0.97, torch.zeros_like(many), many)
    counts = [rs.chunk_total(D, topo) for D in (few, many)]
    a, b = _us(*[_sort(D, topo, n, n) for D, n in zip((few, many), counts)])
    assert a < 0.75 * b, (a, b)                                          # 0.45 to 0.6; 0.75 to 0.95 when every flow went through every pass


def test_counts_of_many_instances_are_read_once():
    few, many = (_matrices(2, 1, B, 65536, 2) for B in (8000, 65536))
    topo = rs.Topo(2, 1, 65536)
    ws = torch.empty(rs.chunk_sort_workspace_bytes(65536, topo), dtype=torch.uint8, device=DEV)
    a, b = _us(*[lambda D=D: rs.chunk_count(D, topo, ws) for D in (few, many)])
    assert b < 6 * a, (a, b)                                             # 17 / 60 us; 165 when every workgroup of the scan added up all counts
