"""Widths without a finite reciprocal and lengths that are no numbers: byte counts over capacities so small
that a load over a capacity overflows on some links and not on others.  The width is infinite then, its
reciprocal zero, and the length of a link that overflows inf * 0.  The definition compares costs with
`<`, so that a path over such a link is never the cheapest, and largest prices with `>`, which passes over
it; every kernel has to choose the same paths."""
import numpy as np
import pytest

from paper_2604_00317_amd import binding as B
from paper_2604_00317_amd import workloads as W
from test_gpu_resident_scatter import FABRICS, circulant
from test_patch import _adaptive, _random, fabric
from test_patch_blocks import SHAPES

pytestmark = pytest.mark.gpu


def _overflowing(t, seed, plans):
    """(csr, demands): byte counts, and capacities scaled so that between a tenth and nine tenths of the links
    overflow if all commodities used all they can reach."""
    rng = np.random.default_rng(seed)
    d = np.floor(rng.pareto(1.1, (plans, t.n_comm)) * 1e4)
    d[:, rng.integers(0, t.n_comm, 2)] = 0.0
    path_comm = np.repeat(np.arange(t.n_comm), np.diff(t.comm_path_ptr))
    use = np.unique(np.stack([np.asarray(t.path_links, dtype=np.int64),
                              np.repeat(path_comm, np.diff(t.path_link_ptr))]), axis=1)
    reach = np.bincount(use[0], weights=d[0][use[1]], minlength=t.n_links) / t.cap
    # seven of ten reached links have reach / cap above the largest double, by up to what they differ
    scale = np.quantile(reach[reach > 0], 0.3) / np.finfo(np.float64).max
    cap = t.cap * scale
    assert cap.min() > np.finfo(np.float64).tiny
    with np.errstate(over="ignore"):
        over = np.isinf(reach[reach > 0] / scale)
    assert 0.1 <= over.mean() <= 0.9
    csr = list(t.csr())
    csr[1] = cap
    return csr, d


def _check(oracle_mod, csr, d, iters, flags, patches=None, regime=0, layout=0):
    n_links = csr[0]
    refs = [oracle_mod.solve(*csr, x, 0.05, iters, flags=flags, len0=np.ones(n_links)) for x in d]
    assert any(np.isnan(r["len"]).any() and np.isfinite(r["len"]).any() for r in refs)
    h = B.nimble_topo_create(*csr, flags=flags | layout)
    try:
        B.nimble_topo_set_regime(h, regime)
        splits, lam = B.plan(h, d, 0.05, iters)
        used = h.last_patches
        for b, ref in enumerate(refs):
            assert np.array_equal(splits.reshape(len(d), -1)[b], ref["splits"]), b
            assert np.atleast_1d(lam)[b] == ref["lam"], b
        if patches is not None:
            assert (used > 1) if patches > 1 else (used == patches)
            assert not B.nimble_debug_patches_gave_up(h)
    finally:
        h.close()
    return refs


@pytest.mark.parametrize("flags", [0, 1])
@pytest.mark.parametrize("lanes", [0, 1, 2, 4])
@pytest.mark.parametrize("strips", [1, 2, 3, 6])
def test_slots(oracle_mod, monkeypatch, strips, lanes, flags):
    monkeypatch.setenv("NIMBLE_TUNE_PATCH_STRIPS", str(strips))
    monkeypatch.setenv("NIMBLE_TUNE_PATCH_LANES", str(lanes))
    monkeypatch.setenv("NIMBLE_TUNE_PATCH_BLOCKS", "0")
    for name in ((2, 8, "pair"), (3, 4, "xor"), (3, 8, "xor"), (8, 4, "own"), (13, 200, 150, 20, 4),
                 (5, 500, 900, 12, 2)):
        t = _random(*name) if len(name) > 3 else fabric(*name)
        there = B.nimble_host_patch_check(t.n_links, t.n_comm, t.comm_path_ptr, t.n_paths, t.path_link_ptr,
                                          t.path_links, strips, lanes)["patches"]
        if there > 0:                                # (no kernel for so many slots in so many lanes)
            print(f"[overflow slots] {name} strips={strips} lanes={lanes} flags={flags}", flush=True)
            _check(oracle_mod, *_overflowing(t, 3, 2), 60, flags, patches=there)


@pytest.mark.parametrize("flags", [0, 1])
@pytest.mark.parametrize("grid", ["2", "4x5", "6"])
@pytest.mark.parametrize("shape", sorted(SHAPES))
def test_blocks(oracle_mod, monkeypatch, shape, grid, flags):
    monkeypatch.setenv("NIMBLE_TUNE_PATCH_STRIPS", grid)
    monkeypatch.setenv("NIMBLE_TUNE_PATCH_BLOCKS", "1")
    print(f"[overflow blocks] {shape} grid={grid} flags={flags}", flush=True)
    _check(oracle_mod, *_overflowing(fabric(*SHAPES[shape]), 4, 2), 60, flags, patches=2)


@pytest.mark.parametrize("nodes,gpus,rails,iters", [(8, 4, "own", 400), (10, 4, "own", 40)])
def test_the_layouts_chosen(oracle_mod, nodes, gpus, rails, iters):
    """What such a call runs on with nothing forced: blocks on several patches."""
    print(f"[overflow chosen] {nodes}x{gpus} {rails}", flush=True)
    _check(oracle_mod, *_overflowing(fabric(nodes, gpus, rails), 5, 1), iters, 0, patches=2)


@pytest.mark.parametrize("blocks", [0, 1])
@pytest.mark.parametrize("flags", [0, 1])
def test_a_warm_start_from_lengths_that_are_no_numbers(oracle_mod, monkeypatch, flags, blocks):
    import torch
    monkeypatch.setenv("NIMBLE_TUNE_PATCH_STRIPS", "3")
    monkeypatch.setenv("NIMBLE_TUNE_PATCH_BLOCKS", str(blocks))
    t = fabric(7, 6, "pair")
    csr, d = _overflowing(t, 6, 2)
    d[1] = np.minimum(d[1], 1.0)                   # a plan of its own has an ordinary width
    length = torch.ones(t.n_links, dtype=torch.float64, device="cuda:0")
    splits = torch.empty(t.n_paths, dtype=torch.float64, device="cuda:0")
    lam = torch.empty(1, dtype=torch.float64, device="cuda:0")
    start = np.ones(t.n_links)
    h = B.nimble_topo_create(*csr, flags=flags)
    try:
        for b in range(2):
            print(f"[overflow warm] flags={flags} blocks={blocks} plan {b}", flush=True)
            B.nimble_plan_solve_warm(h, torch.as_tensor(d[b]).to("cuda:0"), 0.05, 30, length, splits, lam)
            assert h.last_patches > 1 and not B.nimble_debug_patches_gave_up(h)
            ref = oracle_mod.solve(*csr, d[b], 0.05, 30, flags=flags, len0=start)
            assert np.array_equal(splits.cpu().numpy(), ref["splits"]), b
            assert float(lam.item()) == ref["lam"], b
            assert np.array_equal(length.cpu().numpy(), ref["len"], equal_nan=True), b
            start = ref["len"]
    finally:
        h.close()


def test_demands_no_grid_holds(oracle_mod, monkeypatch):
    """One patch, loads added one after the other (a demand so small that no sum of the others moves by it)."""
    monkeypatch.setenv("NIMBLE_TUNE_PATCH_STRIPS", "1")
    csr, d = _overflowing(fabric(2, 8, "pair"), 7, 1)
    d[0] = np.floor(d[0]) + 1.0
    d[0, 100] = 2.0 ** -100
    print("[overflow] one patch, no grid", flush=True)
    _check(oracle_mod, csr, d, 60, 0, patches=1)


@pytest.mark.parametrize("flags", [0, 1])
@pytest.mark.parametrize("where", FABRICS, ids=lambda f: f"{f[0]}{f[1]}")
def test_one_commodity_and_link_per_thread(oracle_mod, where, flags):
    """k_resident_reg, whole bytes and fractions; and capacities without a finite reciprocal on links that
    carry nothing, so that the width is an ordinary number and 0 * inf is the load over a capacity."""
    kind, what = where
    if kind == "node":
        t = W.build_fabric(1, what)
    elif kind == "mesh":
        t = W.two_candidate_mesh(what)
    elif kind == "circulant":
        t = circulant(*what)
    else:
        t = W.random_topology(np.random.default_rng(what[0]), what[1], what[2], what[3], min(2, what[1]))
    print(f"[overflow registers] {where} flags={flags}", flush=True)
    if t.n_links > 1:
        csr, d = _overflowing(t, 8, 3)
        d[2] /= 7.0
        _check(oracle_mod, csr, d, 40, flags)
    rng = np.random.default_rng(9)
    d = np.where(rng.random((2, t.n_comm)) < 0.1, np.floor(rng.random((2, t.n_comm)) * 1e6) + 1.0, 0.0)
    path_comm = np.repeat(np.arange(t.n_comm), np.diff(t.comm_path_ptr))
    reach = np.zeros(t.n_links)
    np.maximum.at(reach, t.path_links, np.repeat(d.max(axis=0)[path_comm], np.diff(t.path_link_ptr)))
    csr = list(t.csr())
    csr[1] = np.where((reach == 0) & (np.arange(t.n_links) % 2 == 0), 1e-310, t.cap)
    if (reach == 0).sum() > 2 and d.any(axis=1).all():
        _check(oracle_mod, csr, d, 40, flags)


@pytest.mark.parametrize("flags", [0, 1])
@pytest.mark.parametrize("layout", [0, 2])
@pytest.mark.parametrize("regime", [B.NIMBLE_REGIME_STREAM, B.NIMBLE_REGIME_PERSISTENT])
def test_streamed(oracle_mod, regime, layout, flags):
    """Record kernels and the reduce kernels of every layout, one plan and three; several waves of a row."""
    for name in ((2, 8, "pair"), (7, 6, "pair"), (3, 8, "xor"), (8, 4, "own"), (5, 500, 900, 12, 2),
                 (13, 200, 150, 20, 4), (16, 300, 700, 40, 7)):
        t = _random(*name) if len(name) > 3 else fabric(*name)
        print(f"[overflow streamed] {name} regime={regime} layout={layout} flags={flags}", flush=True)
        csr, d = _overflowing(t, 10, 3)
        if regime == B.NIMBLE_REGIME_STREAM:
            _check(oracle_mod, csr, d, 30, flags, regime=regime, layout=layout)
        _check(oracle_mod, csr, d[:1], 30, flags, regime=regime, layout=layout)


@pytest.mark.parametrize("flags", [0, 1])
@pytest.mark.parametrize("generic", [False, True])
def test_resident(oracle_mod, monkeypatch, generic, flags):
    """One workgroup per plan: lanes that share commodities, with lists in registers or not, and a thread
    per commodity."""
    monkeypatch.setenv("NIMBLE_TUNE_PATCH_STRIPS", "0")
    if generic:
        monkeypatch.setenv("NIMBLE_TUNE_RESIDENT_GENERIC", "1")
    for name in ((1, 8, "none"), (2, 8, "pair"), (3, 4, "xor"), (13, 200, 150, 20, 4), (5, 500, 900, 12, 2),
                 (20, 100, 90, 20, 5), (18, 60, 80, 3, 4)):
        t = _random(*name) if len(name) > 3 else fabric(*name)
        print(f"[overflow resident] {name} generic={generic} flags={flags}", flush=True)
        csr, d = _overflowing(t, 11, 2)
        _check(oracle_mod, csr, d, 40, flags, regime=B.NIMBLE_REGIME_RESIDENT)


@pytest.mark.parametrize("strips", [0, 1, 3])
@pytest.mark.parametrize("kind", ["all", "few", "capacities"])
def test_variable_step(oracle_mod, monkeypatch, kind, strips):
    """Steps of zero (the largest load over a capacity is infinite): splits stay on the first candidates,
    lambda is 0 / 0, no number, and never below a bound; loads just below the largest double; and
    capacities without a finite reciprocal."""
    monkeypatch.setenv("NIMBLE_TUNE_PATCH_STRIPS", str(strips))
    for name in ((2, 8, "pair"), (3, 4, "xor"), (7, 6, "pair")):
        t = fabric(*name)
        csr, d = _overflowing(t, 3, 1)
        if kind == "few":
            csr[1] = csr[1] * 30.0
        elif kind == "capacities":
            csr[1] = np.where(np.arange(t.n_links) % 5 == 0, 1e-310, t.cap)
        print(f"[overflow adaptive] {name} {kind} strips={strips}", flush=True)
        ref = oracle_mod.solve_adaptive(*csr, d[0], 0.05, 40, 7)
        h = B.nimble_topo_create(*csr)
        try:
            splits, lam, done, lb = _adaptive(h, t, d[0], 0.05, 40, 7)
            assert (done, lb) == (ref["iters"], ref["lb"])
            assert np.array_equal([lam], [ref["lam"]], equal_nan=True)
            assert np.array_equal(splits, ref["splits"])
        finally:
            h.close()
