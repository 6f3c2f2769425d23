"""Register-resident kernel: loads summed by scatter or by gather, against the oracle bit for bit.

The kernel scatters where the demands of a plan lie on a power-of-two grid with a total below
2^52 units and gathers, in the oracle's own order, everywhere else: both are the oracle's bits for
any demands.  Sizes: every instantiation (4 to 8 candidates with a direct first one, 8 with any; each for
plans of one wave and of several), one plan and batches that mix both kinds of demands.
"""
import numpy as np
import pytest

from paper_2604_00317_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a visible MI355X; no fallback path exists")
    from paper_2604_00317_amd import binding
    binding.load_library(build_if_missing=False)
    return binding


def demands_of(kind, K, rng):
    d = np.floor(rng.pareto(1.1, K) * 1e6)
    if kind == "bytes":
        d[rng.integers(0, K)] = 0.0
    elif kind == "zero":
        d[:] = 0.0
    elif kind == "one":
        d[:] = 0.0
        d[K // 2] = 3.0
    elif kind == "fractional":
        d = d / 7.0
    elif kind in ("total_2^51", "total_2^53"):     # either side of the limit of the scatter
        d = np.floor(rng.random(K) * 64)
        d[0] = 1.0
        d[1] = 2.0 ** int(kind[8:]) - 1.0
    elif kind == "denormal":                       # a grid and loads that are denormal
        d = np.floor(rng.random(K) * 1000) * 2.0 ** -1070
    elif kind == "denormal_grid":                  # some demands denormal, a width that is not
        d = np.floor(rng.random(K) * 2.0 ** 44) * 2.0 ** -1030
        d[::3] = np.floor(rng.random(d[::3].size) * 128) * 2.0 ** -1030
    elif kind == "denormal_spread":                # a denormal grid with too large a total
        d = np.floor(rng.random(K) * 1000) * 2.0 ** -1070
        d[0] = 2.0 ** -900
    elif kind == "tiny":                           # a width whose reciprocal is infinite
        d = np.floor(rng.random(K) * 2.0 ** 40) * 2.0 ** -1060
    elif kind == "tiny_spread":
        d = np.floor(rng.random(K) * 1000) * 2.0 ** -1070
        d[0] = 2.0 ** -1000
    elif kind == "tiny_one":                       # the same on a grid that doubles hold
        d[:] = 0.0
        d[K // 2] = 2.0 ** -1020
    elif kind == "huge":
        d = d * 2.0 ** 900
    return d


KINDS = ["bytes", "zero", "one", "fractional", "total_2^51", "total_2^53", "denormal", "denormal_grid",
         "denormal_spread", "tiny", "tiny_spread", "tiny_one", "huge"]
# nodes of 3 to 9 GPUs (2 to 8 candidates, the last with 72 pairs); random topologies of up to 8
# candidates whose first is not always direct: one wave, two waves, a full workgroup's threads; several
# waves with a direct first candidate: meshes (2 candidates), circulant lists of 5 to 8 (of 8 in one too)
FABRICS = [("node", g) for g in (3, 4, 5, 6, 7, 8, 9)] + [
    ("random", (31, 64, 64, 5)), ("random", (32, 130, 100, 8)), ("random", (33, 1024, 700, 4)),
    ("random", (34, 1, 2, 1)), ("mesh", 11), ("mesh", 31), ("circulant", (90, 5)),
    ("circulant", (90, 6)), ("circulant", (90, 7)), ("circulant", (400, 7)), ("circulant", (90, 8)), ("circulant", (60, 8))]


def circulant(n, most):
    """n pairs and links; pair k has its own link, and up to `most` - 1 ways over links k + 2j - 1 and
    k + 2j, so that a link has at most 2 `most` - 1 pairs."""
    cp, lp, pl = [0], [0], []
    for k in range(n):
        pl += [k]
        lp.append(len(pl))
        for j in range(1, most - k % 3 if k else most):
            pl += [(k + 2 * j - 1) % n, (k + 2 * j) % n]
            lp.append(len(pl))
        cp.append(len(lp) - 1)
    cap = np.random.default_rng(n).choice([25.0, 50.0, 100.0], size=n) * 1e9
    zeros = np.zeros(n, dtype=np.int32)
    return W.Topology(n_links=n, cap=cap, n_comm=n, comm_path_ptr=np.asarray(cp, dtype=np.int32),
                      n_paths=len(lp) - 1, path_link_ptr=np.asarray(lp, dtype=np.int32),
                      path_links=np.asarray(pl, dtype=np.int32), src=zeros, dst=zeros,
                      meta=dict(kind="circulant"))


@pytest.mark.parametrize("flags", [0, 1])
@pytest.mark.parametrize("fabric", FABRICS, ids=lambda f: f"{f[0]}{f[1]}")
def test_scatter_and_gather_are_the_oracles_bits(oracle_mod, B, fabric, flags):
    kind, what = fabric
    if kind == "node":
        t = W.build_fabric(1, what)
    elif kind == "mesh":
        t = W.two_candidate_mesh(what)
    elif kind == "circulant":
        t = circulant(*what)
    else:
        seed, E, K, pm = what
        t = W.random_topology(np.random.default_rng(seed), E, K, pm, min(2, E))
    rng = np.random.default_rng(7)
    plans = np.stack([demands_of(k, t.n_comm, rng) for k in KINDS])
    iters = 40
    refs = [oracle_mod.solve(*t.csr(), d, 0.07, iters, flags=flags) for d in plans]
    print(f"{fabric} K={t.n_comm} E={t.n_links} flags={flags}", flush=True)
    h = B.nimble_topo_create(*t.csr(), flags=flags)
    try:
        assert h.resident_in_registers
        splits, lam = B.plan(h, plans, 0.07, iters)             # side by side in a workgroup
        for i, r in enumerate(refs):
            assert np.array_equal(splits[i], r["splits"]) and lam[i] == r["lam"], KINDS[i]
        for i, r in enumerate(refs):
            s, l = B.plan(h, plans[i], 0.07, iters)
            assert np.array_equal(s, r["splits"]) and l == r["lam"], KINDS[i]
    finally:
        h.close()


@pytest.mark.parametrize("iters", [127, 128, 129, 255, 256, 600])
def test_gathered_plans_count_every_iteration(oracle_mod, B, iters):
    """The gather counts choices eight bits at a time: either side of every emptying, and a commodity
    that takes the same candidate on all iterations (a direct link costs half of a detour)."""
    t = W.build_fabric(1, 9)
    rng = np.random.default_rng(iters)
    d = np.stack([demands_of("fractional", t.n_comm, rng) for _ in range(3)])
    d[1, 1:] = 0.0
    d[2] = 1.0 / 3.0
    h = B.nimble_topo_create(*t.csr())
    try:
        splits, lam = B.plan(h, d, 1e-6, iters)        # tiny steps: choices stay for many iterations
        for i in range(3):
            r = oracle_mod.solve(*t.csr(), d[i], 1e-6, iters)
            assert np.array_equal(splits[i], r["splits"]) and lam[i] == r["lam"], i
            sums = np.add.reduceat(splits[i], t.comm_path_ptr[:-1])
            assert np.allclose(sums, 1.0, rtol=0, atol=1e-12)
    finally:
        h.close()
