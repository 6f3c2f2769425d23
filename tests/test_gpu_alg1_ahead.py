"""Algorithm 1 with the loads of a pair read before the pair before it has routed: bit for bit the
oracle's where consecutive pairs fight for the same links, and at the edges of the padded pair loop."""
import numpy as np
import pytest

from paper_2604_00317_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2604_00317_amd import binding
    binding.load_library(build_if_missing=False)
    return binding


def check(oracle_mod, B, t, demands, phi, chi):
    h = B.nimble_topo_create(*t.csr())
    try:
        flows, lam, sweeps = B.plan_alg1(h, demands, phi, chi)
    finally:
        h.close()
    for b in range(demands.shape[0]):
        ref = oracle_mod.alg1(*t.csr(), demands[b], phi, chi)
        assert np.array_equal(flows[b], ref["flows"]), f"problem {b}"
        assert lam[b] == ref["lam"] and sweeps[b] == ref["sweeps"], f"problem {b}"


# (links, pairs, most candidates, most links of a path): two to nine links for all pairs, so that
# most pairs want what the pair before has just loaded; 1 to 16 candidates, pairs around multiples
# of four; then groups of more lanes than the ahead form has, and longer paths
SHAPES = [(2, 1, 2, 2), (2, 2, 2, 1), (3, 3, 1, 2), (3, 4, 3, 2), (4, 5, 4, 2), (9, 56, 7, 2),
          (9, 57, 8, 2), (6, 59, 16, 2), (20, 61, 9, 2), (9, 30, 17, 2), (9, 30, 6, 3), (9, 31, 20, 7)]


@pytest.mark.parametrize("shape", SHAPES, ids=str)
def test_consecutive_pairs_on_the_same_links(oracle_mod, B, shape):
    E, K, pm, lm = shape
    rng = np.random.default_rng(E * 100 + K)
    t = W.random_topology(rng, E, K, pm, lm)
    d = np.floor(rng.pareto(1.1, (21, K)) * 1e6)
    d[1] = 0.0
    d[2, ::2] = 0.0
    d[3] = d[3] / 7.0
    d[4] = np.floor(rng.random(K) * 1000) * 2.0 ** -1070          # denormal bytes, one chunk each
    print(f"[alg1] {shape}", flush=True)
    check(oracle_mod, B, t, d, 0.5, 65536.0)


@pytest.mark.parametrize("gpus,rails", [(8, "own"), (5, "own"), (8, "pair")])
def test_two_nodes(oracle_mod, B, gpus, rails):
    """Long paths on a group of lanes; a NIC per GPU takes more lanes than a pair has candidates."""
    t = W.build_fabric(2, gpus, gpus, [[r] for r in range(gpus)]) if rails == "own" else \
        W.build_fabric(2, gpus, gpus // 2, W.pair_access(gpus // 2))
    rng = np.random.default_rng(gpus)
    d = np.floor(rng.pareto(1.1, (9, t.n_comm)) * 1e6)
    check(oracle_mod, B, t, d, 0.5, float(1 << 20))


def fabric(what):
    if isinstance(what, str):
        nodes, gpus, rails = what.split()
        nodes, gpus = int(nodes), int(gpus)
        if rails == "none":
            return W.build_fabric(nodes, gpus)
        access = W.xor_access(gpus) if rails == "xor" else [[r] for r in range(gpus)]
        return W.build_fabric(nodes, gpus, gpus, access)
    return W.random_topology(np.random.default_rng(5), *what)


# (fabric, problems, kernel: 0 a thread per problem, else 100 x kind + lanes with kind 1 loads read
# ahead, 2 lists in LDS, 3 lists from memory): every kind, at 2, 5 and 8 links of a path, at every
# count of lanes that a rule can give it, and batches on both sides of a change
FORMS = [
    ("1 4 none", 21, 104), ("1 4 none", 65536, 204),
    ("1 10 none", 21, 116), ("1 10 none", 2112, 216), ("1 10 none", 20000, 316),
    ("1 12 none", 21, 116), ("1 12 none", 1500, 316),      # 151 KB of LDS for four problems
    ("1 13 none", 21, 316), ("1 16 none", 21, 316),        # no room for the loads read ahead
    ("2 4 own", 1, 204), ("2 4 own", 21, 204), ("2 4 xor", 21, 216), ("2 4 xor", 16384, 316),
    ("3 4 own", 21, 304),
    ((100, 30, 33, 2), 21, 232), ((200, 60, 8, 8), 21, 208), ((60, 200, 4, 8), 21, 304),
    ((30, 50, 33, 8), 21, 364), ((30, 20, 64, 5), 21, 264), ((30, 20, 64, 5), 8192, 364),
    ((60, 200, 2, 2), 21, 304), ((60, 400, 1, 2), 21, 308),
    ((20, 60, 4, 5), 21, 204), ((20, 60, 4, 5), 65536, 0),
]


@pytest.mark.parametrize("what,batch,form", FORMS, ids=str)
def test_every_form_is_the_oracles_bits(oracle_mod, B, what, batch, form):
    t = fabric(what)
    rng = np.random.default_rng(batch)
    n = min(batch, 21)
    d = np.minimum(np.floor(rng.pareto(1.1, (n, t.n_comm)) * 1e6), 2e7)
    d[-1] = d[-1] / 7.0
    if n > 3:
        d[1] = 0.0                               # nothing to do beside problems that have
        d[2, ::2] = 0.0
        d[3] = np.where(np.arange(t.n_comm) == t.n_comm // 2, 1e8, 0.0)   # one pair, many sweeps
    rows = np.arange(batch) % n
    print(f"[alg1] {what} x {batch}", flush=True)
    h = B.nimble_topo_create(*t.csr())
    try:
        assert h.alg1_form(batch) == form
        flows, lam, sweeps = B.plan_alg1(h, d[rows], 0.5, float(1 << 20))
    finally:
        h.close()
    for i in range(n):
        ref = oracle_mod.alg1(*t.csr(), d[i], 0.5, float(1 << 20))
        assert (flows[rows == i] == ref["flows"]).all(), f"problem {i}"
        assert (lam[rows == i] == ref["lam"]).all() and (sweeps[rows == i] == ref["sweeps"]).all()


def test_more_lds_than_a_kernel_has_by_default_under_capture(oracle_mod, B):
    """The first call on a topology whose groups want more than 64 KB, made while capturing."""
    import torch
    t = fabric("2 6 own")
    rng = np.random.default_rng(3)
    d = np.floor(rng.pareto(1.1, (2, 5, t.n_comm)) * 1e6)
    h = B.nimble_topo_create(*t.csr())
    try:
        assert h.alg1_form(5) == 308
        dd = torch.as_tensor(d[0].reshape(-1)).to("cuda:0")
        ff = torch.zeros(5 * t.n_paths, dtype=torch.float64, device="cuda:0")
        ll = torch.zeros(5, dtype=torch.float64, device="cuda:0")
        ss = torch.zeros(5, dtype=torch.int32, device="cuda:0")
        torch.cuda.synchronize()
        side = torch.cuda.Stream()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            B.nimble_alg1_solve_batch(h, 5, dd, 0.5, 65536.0, 1 << 20, ff, ll, ss,
                                      stream=torch.cuda.current_stream())
        for turn in range(4):
            dd.copy_(torch.as_tensor(d[turn % 2].reshape(-1)))
            ff.fill_(-1.0)
            graph.replay()
            torch.cuda.synchronize()
            got = ff.cpu().numpy().reshape(5, -1)
            for i in range(5):
                ref = oracle_mod.alg1(*t.csr(), d[turn % 2][i], 0.5, 65536.0)
                assert np.array_equal(got[i], ref["flows"]) and ll[i].item() == ref["lam"]
                assert ss[i].item() == ref["sweeps"]
    finally:
        h.close()


def test_topologies_beyond_the_limits_are_refused(B):
    t = W.random_topology(np.random.default_rng(1), 8000, 10, 2, 2)
    h = B.nimble_topo_create(*t.csr())
    try:
        with pytest.raises(B.NimbleError) as e:
            B.plan_alg1(h, np.ones((1, 10)), 0.5, 1.0)
        assert e.value.status == B.NIMBLE_ERR_RANGE
    finally:
        h.close()
