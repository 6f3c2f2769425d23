"""The patch layout in blocks (L commodities with the same tails, their heads kept once) and its
kernels: the layout reads back to the CSR on the CPU, and on the GPU every shape gives the plans of the
oracle, on grids that fit one XCD and on others."""
import numpy as np
import pytest

from paper_2604_00317_amd import binding as B
from test_patch import FABRICS, RANDOM, _random, _topology, direct_mesh, fabric

# ways on from a head (0: one, 1: two) and lanes of a block
SHAPES = {(0, 2): (9, 2, "own"), (0, 4): (8, 4, "own"), (0, 8): (5, 7, "own"),
          (1, 2): (8, 4, "pair"), (1, 4): (6, 6, "pair"), (1, 8): (5, 6, "xor")}


def _check(t, x, y, blocks=1):
    return B.nimble_host_grid_check(t.n_links, t.n_comm, t.comm_path_ptr, t.n_paths, t.path_link_ptr,
                                    t.path_links, x, y, blocks)


@pytest.mark.parametrize("x,y", [(2, 2), (3, 2), (2, 5), (4, 8), (16, 16)])
def test_blocks_read_back(x, y):
    built = 0
    for t in [fabric(*f) for f in FABRICS] + [fabric(*f) for f in SHAPES.values()] + \
            [_random(*r) for r in RANDOM] + [direct_mesh(12)]:
        for blocks in (0, 1):
            s = _check(t, x, y, blocks)
            assert s["failed"] == 0, (t.n_comm, s)
            built += blocks and s["patches"] > 0
    assert built >= 10


def test_every_shape_has_a_fabric():
    for shape, f in SHAPES.items():
        s = _check(fabric(*f), 2, 3)
        assert (s["product"], s["lanes"]) == shape and s["patches"] == 6


def test_heads_and_tails_are_kept_once():
    """One patch row of eight sources against all destinations of another node: as many head blocks as
    rails, whatever the destination; of pairs inside a node nothing is shared."""
    t = fabric(2, 8, "pair")
    s = _check(t, 2, 2)          # a node against a node
    # four rails to the other node (eight sources: two blocks), or 56 pairs in blocks of four
    assert s["max_heads"] == 14 * 4 and s["max_tails"] == 8 * 4 and s["max_comm"] == 64


def test_paths_without_a_middle_keep_their_order():
    """Commodities whose paths have up to five links with and without a link in every place, so that
    the places of a path's links are moved: the candidates read back in order."""
    rng = np.random.default_rng(3)
    lists = []
    for k in range(60):
        paths = []
        for r in range(int(rng.integers(1, 5))):
            full = [10 + k % 7, 30 + r, 40 + r, 50 + r, 60 + k % 5]
            lo, hi = int(rng.integers(0, 2)), 5 - int(rng.integers(0, 2))
            paths.append(full[lo:hi])
        lists.append(paths)
    t = _topology(80, 1e9 + np.arange(80.0), lists)
    for x, y in ((1, 2), (2, 2), (3, 3)):
        s = _check(t, x, y)
        assert s["failed"] == 0, s


def _plan(monkeypatch, t, d, grid, eps, iters, flags=0, spin=None):
    monkeypatch.setenv("NIMBLE_TUNE_PATCH_STRIPS", grid)
    monkeypatch.setenv("NIMBLE_TUNE_PATCH_BLOCKS", "1")
    h = B.nimble_topo_create(*t.csr(), flags=flags)
    try:
        splits, lam = B.plan(h, d, eps, iters)
        return splits, lam, h.last_patches, B.nimble_debug_patches_gave_up(h)
    finally:
        h.close()


@pytest.mark.gpu
@pytest.mark.parametrize("flags", [0, 1])
@pytest.mark.parametrize("grid,patches", [("2", 4), ("3x2", 6), ("4x5", 20), ("6", 36)])
@pytest.mark.parametrize("shape", sorted(SHAPES))
def test_blocks_match_the_oracle(monkeypatch, shape, grid, patches, flags):
    """Byte counts: the oracle's bits; more plans than there are teams, plans without traffic; more
    iterations than 8-bit counters hold."""
    import oracle
    t = fabric(*SHAPES[shape])
    rng = np.random.default_rng(5)
    d = np.floor(rng.pareto(1.1, (9, t.n_comm)) * 1e6)
    d[:, rng.integers(0, t.n_comm, 3)] = 0.0
    d[2] = 0.0
    print(f"[blocks] {shape} {SHAPES[shape]} grid={grid} flags={flags}", flush=True)
    for n, iters in ((9, 17), (1, 300)):
        splits, lam, n_patches, gave_up = _plan(monkeypatch, t, d[:n], grid, 0.05, iters, flags)
        # (a grid finer than the fabric's sources or destinations has fewer patches)
        assert 1 < n_patches <= patches and not gave_up
        for b in range(n):
            ref = oracle.solve(*t.csr(), d[b], 0.05, iters, flags=flags)
            assert np.array_equal(splits[b], ref["splits"]), (shape, b)
            assert lam[b] == ref["lam"], (shape, b)


@pytest.mark.gpu
@pytest.mark.parametrize("grid", ["3", "6"])
def test_fractions_and_wide_demands(monkeypatch, grid):
    """Demands on no common grid: two runs agree bit for bit, and the oracle's sequential sums differ by
    at most one rounding per addition, K * 2^-53 relative, which may turn a tie but moves lambda by less
    than a commodity's choice in one of the iterations does.  Demands that no grid of 105 bits holds are
    given up and solved without patches."""
    import oracle
    t = fabric(6, 6, "pair")
    rng = np.random.default_rng(7)
    d = np.floor(rng.pareto(1.1, t.n_comm) * 1e6) * (1.0 + rng.random(t.n_comm))
    a = _plan(monkeypatch, t, d, grid, 0.05, 40)
    b = _plan(monkeypatch, t, d, grid, 0.05, 40)
    assert a[2] > 1 and not a[3] and a[1] == b[1] and np.array_equal(a[0], b[0])
    ref = oracle.solve(*t.csr(), d, 0.05, 40)
    assert abs(a[1] - ref["lam"]) <= 1e-6 * ref["lam"]
    assert np.mean(a[0] != ref["splits"]) < 0.05
    d = np.floor(d)
    d[3] = 2.0 ** -90
    a = _plan(monkeypatch, t, d, grid, 0.05, 12)
    assert a[3]
    ref = oracle.solve(*t.csr(), d, 0.05, 12)
    assert abs(a[1] - ref["lam"]) <= 1e-9 * ref["lam"]


@pytest.mark.gpu
@pytest.mark.parametrize("grid", ["4", "7"])
def test_a_warm_start_and_a_team_that_cannot_meet(monkeypatch, grid):
    """Lengths handed on from plan to plan; and a limit of zero, at which nobody waits: what the
    patches give up is solved without them."""
    import oracle
    import torch
    t = fabric(7, 6, "pair")
    monkeypatch.setenv("NIMBLE_TUNE_PATCH_STRIPS", grid)
    monkeypatch.setenv("NIMBLE_TUNE_PATCH_BLOCKS", "1")
    rng = np.random.default_rng(8)
    d = np.floor(rng.pareto(1.1, (2, t.n_comm)) * 1e6)
    h = B.nimble_topo_create(*t.csr())
    try:
        length = torch.ones(t.n_links, dtype=torch.float64, device="cuda:0")
        splits = torch.empty(t.n_paths, dtype=torch.float64, device="cuda:0")
        lam = torch.empty(1, dtype=torch.float64, device="cuda:0")
        start = np.ones(t.n_links)
        for b in range(2):
            B.nimble_plan_solve_warm(h, torch.as_tensor(d[b]).to("cuda:0"), 0.05, 20, length, splits, lam)
            assert h.last_patches > 1 and not B.nimble_debug_patches_gave_up(h)
            ref = oracle.solve(*t.csr(), d[b], 0.05, 20, len0=start)
            assert np.array_equal(length.cpu().numpy(), ref["len"]), b
            assert float(lam.item()) == ref["lam"] and np.array_equal(splits.cpu().numpy(), ref["splits"])
            start = ref["len"]
        B.nimble_debug_set_spin_limit(h, 0)
        got = B.plan(h, d[0], 0.05, 20)
        assert B.nimble_debug_patches_gave_up(h)
        ref = oracle.solve(*t.csr(), d[0], 0.05, 20)
        assert got[1] == ref["lam"] and np.array_equal(got[0], ref["splits"])
    finally:
        h.close()
