"""The performance cases of the framework: what one pass through its public entry points costs.

Three families, one dict of plain values per case:

  step      the whole path of one MoE batch: router logits -> top-k and traffic matrix (route_traffic) -> chunks, LPT
            rails, loads (Plan.schedule_one_call).  `batch` is the number of layers planned together: 1 is a layer
            planned when it is reached, 32 or 61 a whole model's layers replayed for planning.
  combine   the second all-to-all of an MoE layer: the traffic matrices transposed, then scheduled.
  flows     traffic matrices that are already known (collected traces, other collectives) scheduled directly, through
            the one call or through the three separate calls with the port choice behind them.

Outputs are integers and are compared exactly.
"""
import math

import torch

import paper_2510_19262_amd as rs

KIB, MIB = 1024, 1024 * 1024
DEV = "cuda"


# ------------------------------------------------------------------------------------------------ cases
def _step(name, M, N, E, k, tokens, batch, payload, chunk, replicas, zipf, gate="fp32", indices=True):
    return {"name": name, "family": "step", "nodes": M, "rails": N, "experts": E, "top_k": k, "tokens_per_gpu": tokens,
            "batch": batch, "payload_bytes": payload, "chunk_bytes": chunk, "replicas": replicas, "zipf": zipf, "gate": gate,
            "indices": indices}


def _flows(name, M, N, batch, chunk, p_zero, median, sigma, call="one", perm=True):
    return {"name": name, "family": "flows", "nodes": M, "rails": N, "batch": batch, "chunk_bytes": chunk, "p_zero": p_zero,
            "median_bytes": median, "sigma": sigma, "call": call, "perm": perm}


def _combine(name, M, N, batch, chunk, tokens, k, payload, zipf, perm=True):
    return {"name": name, "family": "combine", "nodes": M, "rails": N, "batch": batch, "chunk_bytes": chunk,
            "tokens_per_gpu": tokens, "top_k": k, "payload_bytes": payload, "zipf": zipf, "perm": perm}


def listed():
    return [
        # one layer of a small job (4 x 4 GPUs, 8 experts, top-2): launches and host time are all there is
        _step("tiny_layer", 4, 4, 8, 2, 2048, 1, 2 * KIB, 64 * KIB, 2, 1.0),
        # one layer of a decode step on 512 GPUs: 64 tokens a GPU, 256 experts, top-8; almost every flow is a few tokens,
        # shorter than one chunk
        _step("decode_layer", 64, 8, 256, 8, 64, 1, 14 * KIB, 128 * KIB, 4, 1.1),
        # nothing is a power of two: 5 rails, 60 experts, top-6, ragged tokens, 100 000-byte chunks, seven layers
        _step("ragged_layers", 6, 5, 60, 6, 1021, 7, 5 * KIB, 100_000, 1, 0.8),
        # the benchmark workload: 32 layers of 8 experts, top-2, replicated on every node, 16384 tokens a GPU
        _step("prefill_e8", 8, 8, 8, 2, 16384, 32, 8 * KIB, 256 * KIB, 8, 1.2),
        # 16 experts, top-4, one to a GPU: 24 layers of a 16-GPU job
        _step("prefill_e16", 4, 4, 16, 4, 8192, 24, 12 * KIB, 256 * KIB, 1, 1.0),
        # 64 experts, top-6, from a gate that computes in bf16: equal logits are common
        _step("prefill_e64_bf16_gate", 8, 8, 64, 6, 4096, 16, 4 * KIB, 128 * KIB, 1, 0.8, gate="bf16"),
        # one layer of a 512-GPU training step: 256 experts, top-8, 8192 tokens a GPU
        _step("train_layer_e256", 64, 8, 256, 8, 8192, 1, 14 * KIB, 128 * KIB, 4, 1.1),
        # one layer of 512 fine-grained experts, top-10, on 128 GPUs
        _step("train_layer_e512", 16, 8, 512, 10, 4096, 1, 8 * KIB, 128 * KIB, 1, 1.0),
        # the second all-to-all of all 61 layers of the 512-GPU job
        _combine("combine_61_layers", 64, 8, 61, 128 * KIB, 8192, 8, 14 * KIB, 1.1),
        # sparse all-to-all traces on 256 GPUs, heavy-tailed flows, an eighth of the synthetic trace set
        _flows("sparse_traces", 32, 8, 128, 64 * KIB, 0.7, 4 * MIB, 1.5),
        # the same kind of traces through the three separate calls, then the port of every chunk
        _flows("sparse_traces_staged", 32, 8, 32, 64 * KIB, 0.7, 4 * MIB, 1.5, call="staged"),
        # stress: one matrix of 1024 GPUs cut into 16 KiB chunks, about 3.9e9 of them
        _flows("stress_1024_gpus", 128, 8, 1, 16 * KIB, 0.5, 16 * MIB, 2.0, perm=False),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_chunk(rng):
    return rng.choice([16, 32, 64, 128, 256, 512, 1024, 4096]) * KIB if rng.random() < 0.8 else rng.randrange(16_000, 2_000_000)


def _draw_rails(rng):
    return rng.choice([2, 4, 5, 6, 8, 8, 8, 8, 12, 16])


def _draw_step(rng):
    while True:
        N = _draw_rails(rng)
        M = _log_int(rng, 2, 64)
        E = rng.choice([8, 16, 32, 64, 128, 256, 512]) if rng.random() < 0.5 else _log_int(rng, 4, 512)
        k = min(E // 2, rng.choice([1, 2, 2, 4, 6, 8, 8, 10]))
        tokens, batch = _log_int(rng, 16, 16384), _log_int(rng, 1, 48)
        rows = M * N * tokens * batch
        payload = rng.choice([1024, 2048, 2560, 4096, 5120, 6144, 7168]) * 2
        chunk = _draw_chunk(rng)
        G = M * N
        if 4.0 * rows * E > 5e9 or rows * k * payload / chunk + batch * G * G > 3e8 or G > 512 or N * G > 16384:
            continue
        # the indices can be left out where the call makes one pass over the logits
        optional = E <= 8 or (32 < E <= 256 and E % 4 == 0 and k <= 8)
        return dict(_step("", M, N, E, k, tokens, batch, payload, chunk, max(1, min(G // E, rng.choice([1, 1, 2, 4, 8]))),
                          round(rng.uniform(0.0, 1.2), 2), gate=rng.choice(["fp32", "fp32", "bf16"]),
                          indices=not (optional and rng.random() < 0.25)))


def _draw_flows(rng):
    while True:
        N = _draw_rails(rng)
        M, batch = _log_int(rng, 4, 128), _log_int(rng, 1, 256)
        chunk, p_zero, sigma = _draw_chunk(rng), round(rng.uniform(0.0, 0.8), 2), round(rng.uniform(0.5, 2.0), 2)
        c = _flows("", M, N, batch, chunk, p_zero, _log_int(rng, 64 * KIB, 16 * MIB), sigma,
                   call=rng.choice(["one", "one", "staged"]), perm=rng.random() < 0.6)
        if N * M * N <= 16384 and M * N <= 1024 and _flow_chunks(c) < 4e8 and batch * (M * N) ** 2 < 2e7:
            return c


def _draw_combine(rng):
    while True:
        N = _draw_rails(rng)
        M, batch, tokens, k = _log_int(rng, 4, 64), _log_int(rng, 1, 61), _log_int(rng, 16, 16384), rng.choice([1, 2, 4, 6, 8])
        c = _combine("", M, N, batch, _draw_chunk(rng), tokens, k, rng.choice([1024, 2048, 4096, 7168]) * 2,
                     round(rng.uniform(0.0, 1.2), 2), perm=rng.random() < 0.6)
        if N * M * N <= 16384 and M * N <= 512 and _routed_chunks(c) < 4e8:
            return c


def draw(rng):
    u = rng.random()
    c = _draw_step(rng) if u < 0.6 else _draw_flows(rng) if u < 0.85 else _draw_combine(rng)
    del c["name"]
    return c


# ------------------------------------------------------------------------------------------------ what a pass cannot do without
def _flow_chunks(c):
    """Expected chunks of the lognormal flows (all but the intra-node ones)."""
    G = c["nodes"] * c["rails"]
    pairs = c["batch"] * G * (G - c["rails"]) * (1.0 - c["p_zero"])
    return pairs * (c["median_bytes"] * math.exp(c["sigma"] ** 2 / 2) / c["chunk_bytes"] + 0.5)


def _routed_chunks(c):
    """Expected chunks of routed tokens: a source GPU's copies for other nodes spread over the GPUs that hold experts; a flow of
    more than a chunk has half a chunk of tail on average, a shorter one is one chunk."""
    M, N, C = c["nodes"], c["rails"], c["chunk_bytes"]
    G = M * N
    copies = c["tokens_per_gpu"] * c["top_k"] * (1.0 - 1.0 / M)         # of one source GPU, to other nodes
    hosts = min(G, c["experts"] * c["replicas"]) if c["family"] == "step" else G
    hosts *= 1.0 - 1.0 / M
    flows = hosts * (1.0 - math.exp(-copies / hosts))
    return c["batch"] * G * flows * max(1.0, copies * c["payload_bytes"] / (C * flows) + 0.5)


def work(case):
    M, N, B = case["nodes"], case["rails"], case["batch"]
    G = M * N
    perm = case.get("perm", True)
    matrix, loads, offs = 8.0 * B * G * G, 16.0 * B * G + 64.0 * B, 8.0 * (B * M + 1)
    record = 13.0 if perm else 9.0                                    # weight, flow, (perm,) rail
    if case["family"] == "step":
        rows = float(B * G * case["tokens_per_gpu"])
        route = 4.0 * rows * case["experts"] + (4.0 * rows * case["top_k"] if case["indices"] else 0.0) + matrix
        return {"bytes": route + record * _routed_chunks(case) + loads + offs, "flops": 0.0}
    if case["family"] == "combine":
        return {"bytes": 2 * matrix + record * _routed_chunks(case) + loads + offs, "flops": 0.0}
    chunks = _flow_chunks(case)
    # the separate calls hand the records over in memory, and those arrays are inputs of the later calls
    extra = (5.0 + 9.0 + 2.0) - 1.0 if case["call"] == "staged" else 0.0
    return {"bytes": matrix + (record + extra) * chunks + loads + offs, "flops": 0.0}


def tolerance(case):
    return "exact"


# ------------------------------------------------------------------------------------------------ inputs
def _generator(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _popularity(n, s, gen):
    """log of a Zipf(s) popularity over n experts or GPUs, in a seeded order (which one is hot differs by layer and job)."""
    p = -s * torch.log(torch.arange(1, n + 1, device=DEV, dtype=torch.float32))
    return p[torch.randperm(n, device=DEV, generator=gen)]


def _placement(E, G, replicas):
    """int32 [E][replicas]: experts fill a group of GPUs in order, the replicas take further groups."""
    per_gpu = -(-E * replicas // G)
    group = -(-E // per_gpu)
    e = torch.arange(E)[:, None]
    rho = torch.arange(replicas)[None, :]
    return ((rho * group + e // per_gpu) % G).to(torch.int32).contiguous().to(DEV)


def _plan(topo, case, capacity, rows=0, k=0):
    plan = rs.Plan(topo, case["batch"], capacity, DEV, rows=rows, k=k, want_perm=case.get("perm", True))
    for t in (plan.topk_idx, plan.chunk_w, plan.chunk_flow, plan.perm, plan.rail):
        if t is not None:
            t.zero_()                                                  # records behind the last chunk stay defined
    return plan


def prepare(case, seed):
    gen = _generator(seed)
    topo = rs.Topo(case["nodes"], case["rails"], case["chunk_bytes"])
    G, B = topo.G, case["batch"]
    s = {"case": case, "topo": topo}
    if case["family"] == "step":
        E, k, T = case["experts"], case["top_k"], case["tokens_per_gpu"]
        rows = B * G * T
        logits = torch.randn((rows, E), device=DEV, dtype=torch.float32, generator=gen)
        logits += _popularity(E, case["zipf"], gen)
        if case["gate"] == "bf16":
            for part in logits.split(max(1, (1 << 28) // E)):          # in parts: the rounded copy stays small
                part.copy_(part.to(torch.bfloat16))
        # chunks are bounded by the routed bytes and one tail per flow; that is what the record arrays are sized for
        capacity = rows * k * case["payload_bytes"] // case["chunk_bytes"] + min(rows * k, B * G * G) + 1
        s["plan"] = _plan(topo, case, capacity, rows=rows if case["indices"] else 0, k=k)
        s["logits"], s["placement"] = logits, _placement(E, G, case["replicas"])
        s["ws"] = torch.empty(rs.route_traffic_workspace_bytes(B, T, E, k, topo), dtype=torch.uint8, device=DEV)
        return s
    if case["family"] == "combine":
        share = torch.softmax(_popularity(G, case["zipf"], gen), 0)
        mean = (case["tokens_per_gpu"] * case["top_k"] * share).expand(B, G, G)
        D1 = (torch.poisson(mean, generator=gen).to(torch.int64) * case["payload_bytes"]).contiguous()
        s["D1"], s["D1T"] = D1, torch.empty_like(D1)
        # record arrays for the expected bytes and a tail per flow, the same for every seed
        total = B * G * case["tokens_per_gpu"] * case["top_k"] * case["payload_bytes"]
        s["plan"] = _plan(topo, case, int(1.02 * total / case["chunk_bytes"]) + B * G * (G - topo.rails) + 1024)
        return s
    size = torch.randn((B, G, G), device=DEV, dtype=torch.float64, generator=gen)
    size = torch.floor(torch.exp(math.log(case["median_bytes"]) + case["sigma"] * size) / 4096 + 0.5) * 4096
    size.masked_fill_(torch.rand((B, G, G), device=DEV, generator=gen) < case["p_zero"], 0.0)
    size.diagonal(dim1=1, dim2=2).zero_()
    s["D1"] = size.to(torch.int64).contiguous()
    # record arrays for the expected chunks and eight standard deviations of the heavy-tailed flows, the same for every seed
    pairs = max(1.0, B * G * (G - topo.rails) * (1.0 - case["p_zero"]))
    n = int(_flow_chunks(case) * (1.02 + 8.0 * math.sqrt(math.exp(case["sigma"] ** 2) / pairs)) + pairs) + 1024
    s["plan"] = _plan(topo, case, n)
    if case["call"] == "staged":
        s["port"] = torch.zeros(n, dtype=torch.uint8, device=DEV)
    return s


# ------------------------------------------------------------------------------------------------ one pass
def run(state):
    case, topo, plan = state["case"], state["topo"], state["plan"]
    out = {}
    if case["family"] == "step":
        rs.route_traffic(state["logits"], case["top_k"], case["batch"], case["tokens_per_gpu"], state["placement"],
                         case["payload_bytes"], topo, want_idx=case["indices"], out=(plan.topk_idx, plan.D1), ws=state["ws"])
        plan.schedule_one_call()
        out["D1"] = plan.D1
        if case["indices"]:
            out["topk_idx"] = plan.topk_idx
    elif case["family"] == "combine":
        plan.schedule_one_call(rs.transpose_matrix(state["D1"], topo, out=state["D1T"]))
        out["D1T"] = state["D1T"]
    elif case["call"] == "staged":
        plan.schedule(state["D1"])
        out["port"] = rs.port_round_robin(plan.chunk_off, plan.rail, case["batch"], topo, 8, capacity=plan.capacity, out=state["port"])
    else:
        plan.schedule_one_call(state["D1"])
    out.update(chunk_off=plan.chunk_off, chunk_w=plan.chunk_w, chunk_flow=plan.chunk_flow, rail=plan.rail, S=plan.S, R=plan.R,
               stats=plan.stats)
    if plan.perm is not None:
        out["perm"] = plan.perm
    return out
