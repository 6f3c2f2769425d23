"""Timed cases of the planner: what a program that plans All-to-Allv traffic has the library do.

The library is called through `paper_2604_00317_amd.binding`, on modeled fabrics and demand
vectors of `paper_2604_00317_amd.workloads`.  A case names an operation and the fabric, the
traffic and the options it runs on:

    plan      one plan, fixed number of iterations (nimble_plan_solve)
    batch     one plan per MoE layer and micro-batch, all in one call (nimble_plan_solve_batch)
    alg1      the sequential planner of Algorithm 1 on a batch (nimble_alg1_solve_batch)
    warm      a plan that continues from the link lengths of the one before
              (nimble_plan_solve_warm)
    adaptive  variable step, stops on its optimality certificate (nimble_plan_solve_adaptive)
    quantize  split fractions into whole chunks of bytes per path (nimble_plan_quantize)

Fabrics have 1 to 64 nodes of 4 to 8 GPUs; `rails` says how GPUs reach NICs: "none" (one node),
"pair" (GPUs 2r and 2r + 1 share rail r), "xor" (a NIC per GPU, also reachable from the GPU
behind the same switch) or "own" (a NIC per GPU, reachable from that GPU alone).
"""
from __future__ import annotations

from functools import lru_cache

import numpy as np
import torch

from paper_2604_00317_amd import binding as B
from paper_2604_00317_amd import workloads as W

DEVICE = "cuda:0"
CHI = 1 << 20               # chunk of Algorithm 1 and of the quantised plan, bytes
PHI = 0.5                   # fraction of a pair's remainder Algorithm 1 routes per visit
SMALL_MESSAGE = float(1 << 20)
CHECK_EVERY = 25            # iterations between two looks at the adaptive certificate


def _case(op, nodes, gpus, rails, batch=1, eps=0.05, iters=1000, traffic="moe", cost="sum"):
    return dict(op=op, nodes=nodes, gpus=gpus, rails=rails, batch=batch, eps=eps, iters=iters,
                traffic=traffic, cost=cost)


def listed():
    return [
        # the planner inside one node: a single small plan on the critical path of a collective
        dict(_case("plan", 1, 8, "none", eps=0.1, iters=200, traffic="zipf"), name="plan_1x8"),
        # two nodes, the paper's own scale
        dict(_case("plan", 2, 8, "pair", eps=0.1, iters=300), name="plan_2x8"),
        # a fabric that fills no power of two: seven nodes of six GPUs, bottleneck path cost
        dict(_case("plan", 7, 6, "pair", iters=500, cost="max"), name="plan_7x6_bottleneck"),
        # an expert-parallel group of 128 GPUs
        dict(_case("plan", 16, 8, "pair"), name="plan_16x8"),
        # 512 GPUs with a NIC each: the largest fabric
        dict(_case("plan", 64, 8, "xor"), name="plan_64x8"),
        # every MoE layer and micro-batch of a one-node model planned in one call
        dict(_case("batch", 1, 8, "none", batch=4096, eps=0.1, iters=200), name="batch4096_1x8"),
        # the same over two nodes: 61 MoE layers
        dict(_case("batch", 2, 8, "pair", batch=61, eps=0.1, iters=300), name="batch61_2x8"),
        # sixteen micro-batches of the 128-GPU group
        dict(_case("batch", 16, 8, "pair", batch=16), name="batch16_16x8"),
        # the paper's sequential planner on the one-node batch
        dict(_case("alg1", 1, 8, "none", batch=4096), name="alg1_4096_1x8"),
        # replanning every step as traffic drifts: few iterations from the last lengths
        dict(_case("warm", 24, 8, "xor", iters=100), name="warm_24x8"),
        # a plan with a guarantee
        dict(_case("adaptive", 16, 8, "pair", iters=4000), name="adaptive_16x8"),
        # the largest plan handed to a dataplane: bytes per path in whole chunks
        dict(_case("quantize", 64, 8, "xor"), name="quantize_64x8"),
    ]


def _log_int(rng, lo, hi):
    """A whole number from lo to hi, spread evenly over the logarithm."""
    return min(hi, max(lo, int(round(lo * (hi / lo) ** rng.random()))))


def draw(rng):
    op = rng.choice(["plan", "plan", "plan", "batch", "batch", "alg1", "warm", "adaptive",
                     "quantize"])
    gpus = rng.choice([4, 5, 6, 7, 8, 8, 8])
    nodes = _log_int(rng, 1, 64)
    batch = 1
    if op == "batch":
        nodes = _log_int(rng, 1, 24)
        batch = _log_int(rng, 16, 4096) if nodes == 1 else _log_int(rng, 4, 256)
    elif op == "alg1":
        nodes = rng.choice([1, 1, 1, 2])
        batch = _log_int(rng, 64, 4096 if nodes == 1 else 512)
    elif op == "adaptive":
        nodes = _log_int(rng, 2, 24)
    elif op in ("warm", "quantize"):
        nodes = _log_int(rng, 2, 64)
    rails = "none" if nodes == 1 else rng.choice(["pair", "xor", "own"] if gpus % 2 == 0
                                                 else ["own"])
    # no drawn case plans more pairs than the largest listed one
    n_gpus = nodes * gpus
    most = 1000 * 512 * 511 // (n_gpus * (n_gpus - 1))
    if op == "batch":
        batch = max(2, min(batch, most // 100))
    if op in ("plan", "batch"):
        iters = min(_log_int(rng, 100, 1000), most // batch)
    elif op == "warm":
        iters = _log_int(rng, 20, 200)
    elif op == "adaptive":
        iters = _log_int(rng, 300, 1500)
    else:
        iters = 500
    # (the adaptive certificate exists for the additive cost only)
    cost = "max" if op in ("plan", "batch", "warm") and rng.random() < 0.25 else "sum"
    traffic = "zipf" if op != "alg1" and rng.random() < 0.25 else "moe"
    return _case(op, nodes, gpus, rails, batch, rng.choice([0.03, 0.05, 0.1]), iters, traffic,
                 cost)


@lru_cache(maxsize=4)
def _fabric(nodes, gpus, rails):
    """The fabric's arrays on the host: the same for every demand vector planned on it."""
    if rails == "none":
        return W.build_fabric(nodes, gpus)
    if rails == "pair":
        return W.build_fabric(nodes, gpus, gpus // 2, W.pair_access(gpus // 2))
    if rails == "xor":
        return W.build_fabric(nodes, gpus, gpus, W.xor_access(gpus))
    return W.build_fabric(nodes, gpus, gpus, [[r] for r in range(gpus)])


def _traffic(case, topo, rng):
    """Integer byte counts of one demand vector (sizes as in the benchmark configurations)."""
    if case["traffic"] == "zipf":
        return W.zipf_node_traffic(topo, int(rng.integers(1 << 30)))
    experts = 2 * topo.meta["n_nodes"] * topo.meta["gpus_per_node"]
    return W.moe_traffic(topo, 0, tokens=8192, hidden=7168, top_k=min(8, experts // 4),
                         n_experts=experts, s=0.8 + 0.8 * rng.random(), rng=rng)


def prepare(case, seed):
    """Topology handle, demands and output buffers, as a program holds them between plans."""
    topo = _fabric(case["nodes"], case["gpus"], case["rails"])
    op, batch = case["op"], case["batch"]
    flags = B.NIMBLE_COST_MAX if case["cost"] == "max" else B.NIMBLE_COST_SUM
    if op == "batch":
        flags |= B.NIMBLE_LAYOUT_BATCH
    h = B.nimble_topo_create(*topo.csr(), flags=flags)
    if op in ("plan", "warm", "adaptive", "quantize"):
        B.nimble_topo_reserve(h, case["iters"])
    elif op == "batch" and case["nodes"] > 1:
        B.nimble_topo_reserve_batch(h, min(batch, 64), case["iters"])

    rng = np.random.default_rng(seed)
    demands = np.stack([_traffic(case, topo, rng) for _ in range(batch)])
    state = dict(case=case, h=h,
                 traffic=torch.as_tensor(demands.reshape(-1)).to(DEVICE),
                 splits=torch.empty(batch * topo.n_paths, dtype=torch.float64, device=DEVICE),
                 lam=torch.empty(batch, dtype=torch.float64, device=DEVICE))
    if op == "alg1":
        state["sweeps"] = torch.empty(batch, dtype=torch.int32, device=DEVICE)
    elif op == "warm":
        # the lengths the previous plan, for the traffic before it drifted, ended with
        state["last_len"] = torch.ones(topo.n_links, dtype=torch.float64, device=DEVICE)
        before = torch.as_tensor(_traffic(case, topo, rng)).to(DEVICE)
        B.nimble_plan_solve_warm(h, before, case["eps"], case["iters"], state["last_len"],
                                 state["splits"], state["lam"])
        state["len"] = torch.empty_like(state["last_len"])
    elif op == "quantize":
        B.nimble_plan_solve(h, state["traffic"], case["eps"], case["iters"], state["splits"],
                            state["lam"])
        state["flows"] = torch.empty_like(state["splits"])
    return state


def run(state):
    c, h = state["case"], state["h"]
    traffic, splits, lam = state["traffic"], state["splits"], state["lam"]
    op = c["op"]
    if op == "plan":
        B.nimble_plan_solve(h, traffic, c["eps"], c["iters"], splits, lam)
        return splits, lam
    if op == "batch":
        B.nimble_plan_solve_batch(h, c["batch"], traffic, c["eps"], c["iters"], splits, lam)
        return splits, lam
    if op == "alg1":
        B.nimble_alg1_solve_batch(h, c["batch"], traffic, PHI, float(CHI), 1 << 20, splits, lam,
                                  state["sweeps"])
        return splits, lam, state["sweeps"]
    if op == "warm":
        state["len"].copy_(state["last_len"])     # the lengths are updated in place
        B.nimble_plan_solve_warm(h, traffic, c["eps"], c["iters"], state["len"], splits, lam)
        return splits, lam, state["len"]
    if op == "adaptive":
        done, bound = B.nimble_plan_solve_adaptive(h, traffic, c["eps"], c["iters"], CHECK_EVERY,
                                                   splits, lam)
        return splits, lam, done, bound
    B.nimble_plan_quantize(h, traffic, splits, c["iters"], CHI, SMALL_MESSAGE, state["flows"])
    return state["flows"]


def work(case):
    """Bytes: candidate lists, capacities and demands read once, plans written once.  Operations:
    per iteration an addition (or maximum) for every link of every candidate, a comparison per
    candidate, an addition for every link of the chosen candidates and eight operations per
    link; Algorithm 1 counted for the eight sweeps it makes on average; the adaptive step for
    the iterations it needs at least (a quarter of the limit) and its checks."""
    topo = _fabric(case["nodes"], case["gpus"], case["rails"])
    K, P, E, nnz, batch = topo.n_comm, topo.n_paths, topo.n_links, topo.nnz, case["batch"]
    if case["op"] == "quantize":
        return {"bytes": 16 * P + 8 * K + 4 * (K + 1), "flops": 8 * P}
    lists = 4 * (nnz + P + 1 + K + 1) + 8 * E
    per_iter = nnz + P + K * nnz / P + 8 * E
    iters = case["iters"]
    if case["op"] == "alg1":
        iters = 8
    elif case["op"] == "adaptive":
        iters = iters / 4
        per_iter += (K * nnz / P + 2 * K + E) / CHECK_EVERY
    bytes_ = lists + batch * (8 * K + 8 * P + 8)
    if case["op"] == "warm":
        bytes_ += 16 * E
    return {"bytes": bytes_, "flops": batch * iters * per_iter}


def tolerance(case):
    # Demands are whole bytes, so every load sum is exact in any order, and the rest of the
    # arithmetic is defined operation by operation (IEEE binary64, no contraction): plans are the
    # same bits on every correct implementation.
    return "exact"
