"""The insertion kernels of stage 1 at the edges of their shapes (33..1024 logits, k up to 16), against the CPU oracle, exactly:
whole-number outputs, so there is no tolerance."""
import numpy as np
import pytest
import torch

import oracle
import paper_2510_19262_amd as rs

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _bf16(x):
    return torch.from_numpy(x).to(torch.bfloat16).to(torch.float32).numpy()


def _rows(kind, rows, E, rng):
    x = rng.standard_normal((rows, E)).astype(np.float32)
    if kind == "bf16":                               # ties of both signs, nothing lost by the cut
        x = _bf16(x)
    elif kind == "negative":
        x = _bf16(-np.abs(x) - 1)
    elif kind == "close":                            # equal but for the last bits: the cut loses what decides
        base = rng.choice(np.array([2.5, -2.5, 1e-30, -0.0], np.float32), size=(rows, 1))
        x = (base.view(np.int32) + rng.integers(0, 5, size=(rows, E)).astype(np.int32)).view(np.float32)
        x[::2] = rng.standard_normal(x[::2].shape)
    elif kind == "one_lane":                         # all leaders in the places of one lane (float4s E/stride apart)
        for r in range(rows):
            lane = 4 * int(rng.integers(0, 4))
            for c in range(lane, E, 32):
                x[r, c:c + 4] += 10.0
    elif kind == "lowest":                           # masked experts
        x[rng.random((rows, E)) < 0.9] = np.finfo(np.float32).min
    return x


@pytest.mark.parametrize("kind", ["normal", "bf16", "negative", "close", "one_lane", "lowest"])
@pytest.mark.parametrize("E,k", [(36, 1), (64, 6), (64, 8), (68, 7), (128, 8), (132, 8), (256, 8), (256, 3), (260, 1), (260, 9), (512, 8),
                                 (512, 10), (512, 16), (508, 16), (516, 8), (516, 16), (1024, 8), (1024, 10), (1024, 16), (512, 17), (514, 10)])
def test_topk_lists(E, k, kind):
    rng = np.random.default_rng(E * 31 + k)
    for rows in (1, 517):
        x = _rows(kind, rows, E, rng)
        got = rs.route_topk(torch.from_numpy(x).to(DEV), k).cpu().numpy()
        assert np.array_equal(got, oracle.route_topk(x, k))


@pytest.mark.parametrize("k,R,tok", [(6, 1, 4096), (6, 4, 1021), (3, 3, 1000), (10, 1, 77), (5, 2, 4099), (8, 1, 512), (8, 5, 300), (8, 2, 513)])
def test_traffic_matrix_replicas(k, R, tok):
    # slots whose token index needs a division, whose replica index does not, and both
    rng = np.random.default_rng(k * 100 + R)
    E, M, N = 24, 3, 4
    idx = rng.integers(0, E, size=(2 * M * N * tok, k)).astype(np.int32)
    eg = rng.integers(0, M * N, size=(E, R)).astype(np.int32)
    got = rs.traffic_matrix(torch.from_numpy(idx).to(DEV), 2, tok, torch.from_numpy(eg).to(DEV), 2048, rs.Topo(M, N, 65536))
    assert np.array_equal(got.cpu().numpy(), oracle.traffic_matrix(idx, 2, tok, eg, 2048, M, N))


@pytest.mark.parametrize("kind", ["normal", "bf16", "close", "lowest"])
@pytest.mark.parametrize("E,k", [(12, 1), (12, 4), (16, 4), (16, 5), (16, 8), (20, 2), (28, 8), (32, 3), (32, 8), (32, 9), (18, 4)])
def test_one_pass_routing_of_short_rows(E, k, kind):
    rng = np.random.default_rng(E * 17 + k)
    M, N, B, R = 2, 3, 2, 2
    G = M * N
    topo = rs.Topo(M, N, 65536)
    eg = rng.integers(0, G, size=(E, R)).astype(np.int32)
    for tok in (1, 255, 511, 1025):
        x = _rows(kind, B * G * tok, E, rng)
        idx, D1 = rs.route_traffic(torch.from_numpy(x).to(DEV), k, B, tok, torch.from_numpy(eg).to(DEV), 512, topo)
        want = oracle.route_topk(x, k)
        assert np.array_equal(idx.cpu().numpy(), want)
        assert np.array_equal(D1.cpu().numpy(), oracle.traffic_matrix(want, B, tok, eg, 512, M, N))


def _routed(E, k, M, N, B, tok, R=1, ws=None, want_idx=True, x=None, seed=5):
    """One call of route_traffic and the oracle's two stages on the same rows."""
    rng = np.random.default_rng(seed)
    if x is None:
        x = rng.standard_normal((B * M * N * tok, E)).astype(np.float32)
    eg = rng.integers(0, M * N, size=(E, R)).astype(np.int32)
    idx, D1 = rs.route_traffic(torch.from_numpy(x).to(DEV), k, B, tok, torch.from_numpy(eg).to(DEV), 512, rs.Topo(M, N, 65536), ws=ws,
                               want_idx=want_idx)
    want = oracle.route_topk(x, k)
    if want_idx:
        assert np.array_equal(idx.cpu().numpy(), want)
    assert np.array_equal(D1.cpu().numpy(), oracle.traffic_matrix(want, B, tok, eg, 512, M, N))


def test_one_pass_routing_without_room_for_slice_counts():
    # rows of 16 logits with a workspace that only the two stages fit: the same outputs
    M, N, B, E, k, tok = 2, 2, 1, 16, 2, 2100
    topo = rs.Topo(M, N, 65536)
    ws = torch.empty(16, dtype=torch.uint8, device=DEV)
    assert rs.route_traffic_workspace_bytes(B, tok, E, k, topo) > 256 > ws.numel()           # the one pass takes slices here ...
    assert rs.traffic_matrix_workspace_bytes(B, tok, k, topo) == 256                         # ... and the two stages one
    _routed(E, k, M, N, B, tok, ws=ws)


def test_routing_with_room_for_longer_slices_only():
    # rows of 64 logits without indices: half the workspace of the query still holds the counts of slices twice as long, less does not
    M, N, E, k, tok = 8, 8, 64, 6, 512
    need = rs.route_traffic_workspace_bytes(1, tok, E, k, rs.Topo(M, N, 65536))
    assert need == 4 * 64 * 4 * 64                                                           # 64 pairs, 4 slices, 64 counts
    _routed(E, k, M, N, 1, tok, ws=torch.empty(need // 2, dtype=torch.uint8, device=DEV), want_idx=False)
    with pytest.raises(rs.RailschedError):
        _routed(E, k, M, N, 1, tok, ws=torch.empty(need // 2 - 4, dtype=torch.uint8, device=DEV), want_idx=False)
    # rows of 8 logits: few pairs of up to 2048 tokens may stay whole
    assert rs.route_traffic_workspace_bytes(1, 2048, 8, 8, rs.Topo(4, 4, 65536)) > 256
    _routed(8, 8, 4, 4, 1, 2048, ws=torch.empty(256, dtype=torch.uint8, device=DEV))


@pytest.mark.parametrize("E,k,M,N,tok", [(16, 1, 2, 3, 512), (16, 3, 2, 3, 513), (12, 2, 2, 3, 1024), (16, 6, 2, 3, 1025), (12, 8, 2, 2, 2100),
                                         (16, 4, 16, 16, 1025), (16, 7, 16, 16, 2049), (32, 1, 2, 3, 256), (32, 5, 2, 3, 257), (28, 6, 2, 3, 512),
                                         (20, 1, 2, 3, 513), (32, 2, 8, 8, 300), (32, 4, 16, 16, 700)])
def test_slices_of_short_rows(E, k, M, N, tok):
    # rounds of 256 and of 512 threads, one slice and several, one round a slice and more (large G); every width of index stores
    _routed(E, k, M, N, 1, tok, R=2)


@pytest.mark.parametrize("k", [1, 2, 3, 4, 6, 8])
@pytest.mark.parametrize("shift", [1, 2])
def test_index_arrays_at_any_alignment(k, shift):
    # indices behind the first `shift` words of an allocation: 4 and 8 bytes off a 16-byte boundary
    rng = np.random.default_rng(k)
    M, N, E, tok = 2, 2, 16, 600
    rows = M * N * tok
    x = rng.standard_normal((rows, E)).astype(np.float32)
    eg = rng.integers(0, M * N, size=(E, 1)).astype(np.int32)
    room = torch.full((rows * k + 8,), -7, dtype=torch.int32, device=DEV)
    idx = room[shift:shift + rows * k].view(rows, k)
    D1 = torch.empty((1, M * N, M * N), dtype=torch.int64, device=DEV)
    rs.route_traffic(torch.from_numpy(x).to(DEV), k, 1, tok, torch.from_numpy(eg).to(DEV), 512, rs.Topo(M, N, 65536), out=(idx, D1))
    want = oracle.route_topk(x, k)
    assert np.array_equal(idx.cpu().numpy(), want)
    assert (room[:shift] == -7).all() and (room[shift + rows * k:] == -7).all()
    assert np.array_equal(D1.cpu().numpy(), oracle.traffic_matrix(want, 1, tok, eg, 512, M, N))


@pytest.mark.parametrize("E,k,R,tok", [(16, 4, 600, 700), (16, 1, 1000, 1100), (32, 8, 300, 300), (32, 3, 513, 600), (8, 2, 1500, 513), (8, 2, 1500, 2048),
                                       (4, 1, 3000, 1999)])
def test_placement_tables_in_global_memory(E, k, R, tok):
    # more than 8192 entries: the one-pass kernels of up to 8 and of 9..32 logits read the table where it is
    _routed(E, k, 2, 3, 1, tok, R=R)


@pytest.mark.parametrize("E,k,M,N,tok", [(8, 4, 2, 3, 2048), (8, 5, 2, 3, 2048), (8, 8, 2, 3, 1024), (8, 8, 2, 3, 1025), (8, 2, 16, 16, 600), (4, 2, 16, 32, 1100),
                                         (8, 1, 13, 40, 1100)])
def test_whole_pairs_of_rows_of_eight(E, k, M, N, tok):
    # cut or whole by tokens and picks, 256 or 1024 threads by pairs (256, 512 and 520 of them)
    _routed(E, k, M, N, 1, tok)


@pytest.mark.parametrize("E,k,M,N,B,tok", [(64, 2, 2, 2, 1, 20_000), (128, 8, 2, 2, 1, 8300), (256, 2, 2, 2, 1, 4200), (192, 8, 2, 3, 1, 700),
                                           (64, 6, 16, 16, 1, 1537), (96, 4, 8, 8, 2, 1500), (256, 8, 8, 8, 40, 65), (36, 1, 3, 3, 2, 129)])
def test_one_pass_without_indices(E, k, M, N, B, tok):
    # more rows than 128 slices of the shortest length, slices that do not divide the tokens, longer slices for many pairs
    _routed(E, k, M, N, B, tok, want_idx=False)


@pytest.mark.parametrize("E,k,edge", [(512, 1, 8192), (512, 8, 4096), (260, 3, 4096), (516, 2, 16384), (1024, 4, 8192), (768, 16, 4096), (192, 8, 16384),
                                      (240, 2, 16384)])
def test_topk_around_the_row_counts_where_the_kernel_changes(E, k, edge):
    rng = np.random.default_rng(E + k)
    x = _rows("normal", edge + 1, E, rng)
    x[::3] = _bf16(x[::3])
    xd = torch.from_numpy(x).to(DEV)
    want = oracle.route_topk(x, k)
    for rows in (edge, edge + 1):
        assert np.array_equal(rs.route_topk(xd[:rows], k).cpu().numpy(), want[:rows])


@pytest.mark.parametrize("E,tok", [(8, 512), (8, 513), (8, 2048), (8, 2049), (4, 1537), (60, 682), (60, 683), (60, 2730), (60, 2731)])
def test_slices_of_few_pairs(E, tok):
    # around the token counts where a pair's tokens become slices: one workgroup's rounds, or counts summed by a second kernel
    rng = np.random.default_rng(E * 10_000 + tok)
    M, N, k = 2, 3, 2 if E <= 8 else 6
    x = rng.standard_normal((M * N * tok, E)).astype(np.float32)
    eg = rng.integers(0, M * N, size=(E, 2)).astype(np.int32)
    idx, D1 = rs.route_traffic(torch.from_numpy(x).to(DEV), k, 1, tok, torch.from_numpy(eg).to(DEV), 512, rs.Topo(M, N, 65536))
    want = oracle.route_topk(x, k)
    assert np.array_equal(idx.cpu().numpy(), want)
    assert np.array_equal(D1.cpu().numpy(), oracle.traffic_matrix(want, 1, tok, eg, 512, M, N))
