"""The patch layout (commodities cut into patches, one workgroup each) and its kernels: the layout
reads back to the CSR on the CPU, and on the GPU every shape -- slots of either form, one to four
lanes per commodity, one patch and several -- gives the oracle's plans."""
import numpy as np
import pytest

from paper_2604_00317_amd import binding as B
from paper_2604_00317_amd import workloads as W


def fabric(nodes, gpus, rails):
    if nodes == 1:
        return W.build_fabric(1, gpus)
    if rails == "pair":
        return W.build_fabric(nodes, gpus, gpus // 2, W.pair_access(gpus // 2))
    if rails == "xor":
        return W.build_fabric(nodes, gpus, gpus, W.xor_access(gpus))
    return W.build_fabric(nodes, gpus, gpus, [[r] for r in range(gpus)])


FABRICS = [(1, 4, "none"), (2, 8, "pair"), (2, 5, "own"), (3, 4, "xor"), (7, 6, "pair"),
           (4, 8, "own"), (3, 8, "xor")]
RANDOM = [(1, 7, 3, 4, 3), (2, 40, 130, 9, 5), (3, 64, 65, 30, 4), (4, 1, 5, 1, 1),
          (5, 500, 1500, 12, 2)]


def _topology(links, caps, lists):
    """A topology from per-commodity lists of candidate paths (lists of link ids)."""
    cp = np.cumsum([0] + [len(c) for c in lists]).astype(np.int32)
    paths = [p for c in lists for p in c]
    lp = np.cumsum([0] + [len(p) for p in paths]).astype(np.int32)
    pl = np.array([e for p in paths for e in p], dtype=np.int32)
    k = len(lists)
    return W.Topology(n_links=links, cap=np.asarray(caps, dtype=np.float64), n_comm=k,
                      comm_path_ptr=cp, n_paths=len(paths), path_link_ptr=lp, path_links=pl,
                      src=np.zeros(k, dtype=np.int32), dst=np.zeros(k, dtype=np.int32),
                      meta=dict(kind="lists"))


def direct_mesh(gpus):
    """Every pair has one link of its own: patches that share nothing."""
    k = gpus * (gpus - 1)
    return _topology(k, 1e9 * (1 + np.arange(k) % 5), [[[e]] for e in range(k)])


def islands(n, t):
    """n copies of a fabric without links between them."""
    one = [[[int(e) for e in t.path_links[t.path_link_ptr[p]:t.path_link_ptr[p + 1]]]
            for p in range(t.comm_path_ptr[k], t.comm_path_ptr[k + 1])] for k in range(t.n_comm)]
    return _topology(n * t.n_links, np.tile(t.cap, n),
                     [[[e + i * t.n_links for e in p] for p in c] for i in range(n) for c in one])


def _random(seed, E, K, pm, lm):
    return W.random_topology(np.random.default_rng(seed), E, K, pm, lm)


@pytest.mark.parametrize("lanes", [0, 1, 2, 4])
@pytest.mark.parametrize("strips", [1, 2, 3])
def test_layout_reads_back(strips, lanes):
    built = 0
    for t in [fabric(*f) for f in FABRICS] + [_random(*r) for r in RANDOM]:
        s = B.nimble_host_patch_check(t.n_links, t.n_comm, t.comm_path_ptr, t.n_paths,
                                      t.path_link_ptr, t.path_links, strips, lanes)
        assert s["failed"] == 0, (t.n_comm, s)
        built += s["patches"] > 0
    assert built >= 6
    # more candidates than slots hold, and paths of more than five links
    for t in (_random(6, 50, 40, 127, 2), _random(7, 60, 40, 5, 9)):
        assert np.diff(t.comm_path_ptr).max() > 32 or np.diff(t.path_link_ptr).max() > 5
        assert B.nimble_host_patch_check(t.n_links, t.n_comm, t.comm_path_ptr, t.n_paths,
                                         t.path_link_ptr, t.path_links, 1)["patches"] == 0


def _solve(t, d, eps, iters, flags):
    h = B.nimble_topo_create(*t.csr(), flags=flags)
    try:
        out = B.plan(h, d, eps, iters)
        return out[0], out[1], h.regime
    finally:
        h.close()


@pytest.mark.gpu
@pytest.mark.parametrize("flags", [0, 1])
@pytest.mark.parametrize("strips,lanes", [(1, 1), (1, 2), (1, 4), (2, 1), (2, 4), (3, 0), (3, 2)])
def test_patch_kernels_match_the_oracle(monkeypatch, strips, lanes, flags):
    """Byte counts: the same bits as the oracle, whatever the cut; more iterations than 8-bit
    counters hold; a batch with a plan of no traffic."""
    import oracle
    monkeypatch.setenv("NIMBLE_TUNE_PATCH_STRIPS", str(strips))
    monkeypatch.setenv("NIMBLE_TUNE_PATCH_LANES", str(lanes))
    cases = [(f, fabric(*f)) for f in FABRICS[1:]] + [(r, _random(*r)) for r in RANDOM]
    for name, t in cases:
        rng = np.random.default_rng(5)
        d = np.floor(rng.pareto(1.1, (3, t.n_comm)) * 1e6)
        d[:, rng.integers(0, t.n_comm, 3)] = 0.0
        d[2] = 0.0
        print(f"[patch] {name} strips={strips} lanes={lanes} flags={flags}", flush=True)
        iters = 300 if t.n_comm < 300 else 40
        splits, lam, _ = _solve(t, d, 0.05, iters, flags)
        for b in range(3):
            ref = oracle.solve(*t.csr(), d[b], 0.05, iters, flags=flags)
            assert np.array_equal(splits[b], ref["splits"]), (name, b)
            assert lam[b] == ref["lam"], (name, b)


@pytest.mark.gpu
@pytest.mark.parametrize("strips", [1, 3])
def test_fractional_demands_are_deterministic(monkeypatch, strips):
    """Demands on no common grid: a patch sums its loads as integers and rounds when it puts their
    two halves together, so two runs agree bit for bit; the oracle's sequential sums differ from
    them by at most one rounding per addition, K * 2^-53 relative, which may turn a tie but moves
    lambda by less than a commodity's choice in one of the iterations does."""
    import oracle
    monkeypatch.setenv("NIMBLE_TUNE_PATCH_STRIPS", str(strips))
    for f in FABRICS[1:5]:
        t = fabric(*f)
        rng = np.random.default_rng(8)
        d = np.floor(rng.pareto(1.1, t.n_comm) * 1e6) * (1.0 + rng.random(t.n_comm))
        print(f"[patch] fractional {f} strips={strips}", flush=True)
        a = _solve(t, d, 0.05, 60, 0)
        b = _solve(t, d, 0.05, 60, 0)
        assert np.array_equal(a[0], b[0]) and a[1] == b[1]
        ref = oracle.solve(*t.csr(), d, 0.05, 60)
        assert abs(a[1] - ref["lam"]) <= 1e-6 * ref["lam"]
        assert np.mean(a[0] != ref["splits"]) < 0.05


def _adaptive(h, t, d, eps, iters, every):
    import torch
    splits = torch.full((t.n_paths,), float("nan"), dtype=torch.float64, device="cuda:0")
    lam = torch.full((1,), float("nan"), dtype=torch.float64, device="cuda:0")
    done, lb = B.nimble_plan_solve_adaptive(h, torch.as_tensor(d).to("cuda:0"), eps, iters, every,
                                            splits, lam)
    return splits.cpu().numpy(), float(lam.item()), done, lb


@pytest.mark.gpu
@pytest.mark.parametrize("strips,lanes", [(1, 1), (1, 4), (2, 2), (3, 0)])
def test_variable_step_matches_the_oracle(monkeypatch, strips, lanes):
    """The solve of variable step in one launch: the oracle's bits, its stop iteration and bound,
    with checks every iteration, never, and on the last; sums of 1, 255..257 and more terms (1x4:
    12, 3x4 xor: 132, 2x8: 240, 2x9: 306 pairs); no traffic; links no candidate uses; several
    solves with one handle; solved kernel by kernel as well."""
    import oracle
    monkeypatch.setenv("NIMBLE_TUNE_PATCH_STRIPS", str(strips))
    monkeypatch.setenv("NIMBLE_TUNE_PATCH_LANES", str(lanes))
    cases = [(f, fabric(*f)) for f in FABRICS + [(2, 9, "own")]] + \
            [(r, _random(*r)) for r in RANDOM + [(8, 300, 256, 6, 3), (9, 257, 257, 3, 2)]]
    for name, t in cases:
        d = np.floor(np.random.default_rng(3).pareto(1.1, t.n_comm) * 1e6)
        h = B.nimble_topo_create(*t.csr())
        try:
            for iters, every in ((1, 1), (40, 1), (41, 7), (30, 31), (300, 25)):
                print(f"[patch adaptive] {name} strips={strips} lanes={lanes} {iters}/{every}",
                      flush=True)
                ref = oracle.solve_adaptive(*t.csr(), d, 0.1, iters, every)
                for one_launch in (True, False):
                    B.nimble_topo_set_regime(h, 0 if one_launch else B.NIMBLE_REGIME_STREAM)
                    splits, lam, done, lb = _adaptive(h, t, d, 0.1, iters, every)
                    assert (h.last_patches > 0) <= one_launch
                    assert (done, lb, lam) == (ref["iters"], ref["lb"], ref["lam"]), (name, iters)
                    assert np.array_equal(splits, ref["splits"]), (name, iters)
                B.nimble_topo_set_regime(h, 0)
            ref = oracle.solve_adaptive(*t.csr(), 0 * d, 0.1, 9, 1)
            splits, lam, done, lb = _adaptive(h, t, 0 * d, 0.1, 9, 1)
            assert (done, lb, lam) == (0, 0.0, 0.0) and np.array_equal(splits, ref["splits"])
        finally:
            h.close()


@pytest.mark.gpu
def test_a_team_that_cannot_meet_gives_up(monkeypatch):
    """A poll limit of zero: patches that have to wait for each other abandon the solve; lambda is
    right all the same (see test_what_patches_give_up_is_solved_without_them), and the topology
    works again afterwards."""
    import oracle
    monkeypatch.setenv("NIMBLE_TUNE_PATCH_STRIPS", "3")
    t = fabric(7, 6, "pair")
    d = np.floor(np.random.default_rng(9).pareto(1.1, t.n_comm) * 1e6)
    ref = oracle.solve(*t.csr(), d, 0.05, 30)
    h = B.nimble_topo_create(*t.csr())
    try:
        B.nimble_debug_set_spin_limit(h, 0)
        _, lam = B.plan(h, d, 0.05, 30)
        assert np.isnan(lam) or lam == ref["lam"]
        B.nimble_debug_set_spin_limit(h, 1 << 22)
        splits, lam = B.plan(h, d, 0.05, 30)
        assert lam == ref["lam"] and np.array_equal(splits, ref["splits"])
    finally:
        h.close()


@pytest.mark.gpu
def test_phases_can_be_timed_after_a_solve_in_one_launch():
    """The patch kernels leave the streaming workspace alone: the phases set it up themselves, a
    topology that solved nothing is still refused, and plans are the same afterwards."""
    import torch
    t = fabric(7, 6, "pair")
    d = np.floor(np.random.default_rng(9).pareto(1.1, t.n_comm) * 1e6)
    dd = torch.as_tensor(d).to("cuda:0")
    h = B.nimble_topo_create(*t.csr())
    try:
        with pytest.raises(B.NimbleError):
            B.nimble_debug_run_phase(h, 0, 1, dd)
        splits, lam = B.plan(h, d, 0.05, 30)
        for phase in (1, 0, 1):
            B.nimble_debug_run_phase(h, phase, 2, dd)
        torch.cuda.synchronize()
        again, lam2 = B.plan(h, d, 0.05, 30)
        assert lam == lam2 and np.array_equal(splits, again)
    finally:
        h.close()


def test_patches_without_a_shared_link():
    """Fabrics the library cuts into several patches that have nothing to exchange but the width."""
    for t, strips in ((direct_mesh(64), 4), (islands(40, W.build_fabric(1, 8)), 3), (direct_mesh(64), 6),
                      (islands(40, W.build_fabric(1, 8)), 6)):
        s = B.nimble_host_patch_check(t.n_links, t.n_comm, t.comm_path_ptr, t.n_paths,
                                      t.path_link_ptr, t.path_links, strips)
        assert s["failed"] == 0 and s["patches"] > 1 and s["parts"] == 0, s


@pytest.mark.gpu
@pytest.mark.parametrize("flags", [0, 1])
@pytest.mark.parametrize("strips", [0, 4, 6])
def test_patches_without_a_shared_link_match_the_oracle(monkeypatch, strips, flags):
    """What patches meet over is cleared before every solve although no part of a link's load is
    exchanged: solves in a row with one handle (lambda starts as NaN), a batch, a warm start, a
    variable step."""
    import oracle
    import torch
    if strips:
        monkeypatch.setenv("NIMBLE_TUNE_PATCH_STRIPS", str(strips))
    for name, t in (("mesh", direct_mesh(64)), ("islands", islands(40, W.build_fabric(1, 8)))):
        print(f"[patch] {name} strips={strips} flags={flags}", flush=True)
        d = np.floor(np.random.default_rng(11).pareto(1.1, (4, t.n_comm)) * 1e6)
        d[2] = 0.0
        ref = [oracle.solve(*t.csr(), d[b], 0.05, 20, flags=flags) for b in range(4)]
        h = B.nimble_topo_create(*t.csr(), flags=flags)
        try:
            dd = torch.as_tensor(d).to("cuda:0")
            splits = torch.empty((4, t.n_paths), dtype=torch.float64, device="cuda:0")
            lam = torch.full((4,), float("nan"), dtype=torch.float64, device="cuda:0")
            for b in (0, 1, 2, 3, 0):
                lam.fill_(float("nan"))
                B.nimble_plan_solve(h, dd[b], 0.05, 20, splits[b], lam[b:b + 1])
                assert float(lam[b].item()) == ref[b]["lam"], (name, b)
                assert np.array_equal(splits[b].cpu().numpy(), ref[b]["splits"]), (name, b)
            lam.fill_(float("nan"))
            B.nimble_plan_solve_batch(h, 4, dd.reshape(-1), 0.05, 20, splits.reshape(-1), lam)
            assert lam.cpu().numpy().tolist() == [r["lam"] for r in ref]
            for b in range(4):
                assert np.array_equal(splits[b].cpu().numpy(), ref[b]["splits"]), (name, b)
            ln = torch.ones(t.n_links, dtype=torch.float64, device="cuda:0")
            B.nimble_plan_solve_warm(h, dd[1], 0.05, 20, ln, splits[0], lam[:1])
            warm = oracle.solve(*t.csr(), d[1], 0.05, 20, flags=flags, len0=np.ones(t.n_links))
            assert float(lam[0].item()) == warm["lam"]
            assert np.array_equal(ln.cpu().numpy(), warm["len"])
            if not flags:
                a = oracle.solve_adaptive(*t.csr(), d[3], 0.1, 40, 7)
                got = _adaptive(h, t, d[3], 0.1, 40, 7)
                assert got[1:] == (a["lam"], a["iters"], a["lb"])
                assert np.array_equal(got[0], a["splits"])
        finally:
            h.close()


@pytest.mark.gpu
@pytest.mark.parametrize("flags", [0, 1])
def test_what_patches_give_up_is_solved_without_them(monkeypatch, flags):
    """Nobody waits (limit zero): a plan, a batch of more plans than teams, a warm start (whose
    lengths come back whole) and a variable step still give the oracle's bits, as they do with the
    ordinary limit before and after; a fabric of one patch has no waits to give up."""
    import oracle
    import torch
    monkeypatch.setenv("NIMBLE_TUNE_PATCH_STRIPS", "3")
    for t in (fabric(7, 6, "pair"), fabric(3, 8, "xor"), _random(5, 500, 1500, 12, 2)):
        n = 70
        rng = np.random.default_rng(9)
        d = np.floor(rng.pareto(1.1, (n, t.n_comm)) * 1e6)
        d[3] = 0.0
        ref = [oracle.solve(*t.csr(), d[b], 0.05, 5, flags=flags) for b in range(n)]
        len0 = 1.0 + rng.random(t.n_links)
        warm = oracle.solve(*t.csr(), d[1], 0.05, 9, flags=flags, len0=len0)
        h = B.nimble_topo_create(*t.csr(), flags=flags)
        try:
            dd = torch.as_tensor(d).to("cuda:0")
            splits = torch.empty((n, t.n_paths), dtype=torch.float64, device="cuda:0")
            lam = torch.empty(n, dtype=torch.float64, device="cuda:0")
            for limit in (1 << 22, 0, 1 << 22):
                print(f"[patch] gives up K={t.n_comm} flags={flags} limit={limit}", flush=True)
                B.nimble_debug_set_spin_limit(h, limit)
                s, l = B.plan(h, d[0], 0.05, 5)
                assert B.nimble_debug_patches_gave_up(h) == (limit == 0)
                assert l == ref[0]["lam"] and np.array_equal(s, ref[0]["splits"])
                B.nimble_plan_solve_batch(h, n, dd.reshape(-1), 0.05, 5, splits.reshape(-1), lam)
                assert B.nimble_debug_patches_gave_up(h) == (limit == 0)
                assert lam.cpu().numpy().tolist() == [r["lam"] for r in ref]
                for b in range(n):
                    assert np.array_equal(splits[b].cpu().numpy(), ref[b]["splits"]), b
                ln = torch.as_tensor(len0).to("cuda:0")
                B.nimble_plan_solve_warm(h, dd[1], 0.05, 9, ln, splits[0], lam[:1])
                assert B.nimble_debug_patches_gave_up(h) == (limit == 0)
                assert float(lam[0].item()) == warm["lam"]
                assert np.array_equal(ln.cpu().numpy(), warm["len"])
                assert np.array_equal(splits[0].cpu().numpy(), warm["splits"])
                if not flags:
                    a = oracle.solve_adaptive(*t.csr(), d[2], 0.1, 30, 4)
                    got = _adaptive(h, t, d[2], 0.1, 30, 4)
                    assert B.nimble_debug_patches_gave_up(h) == (limit == 0)
                    assert got[1:] == (a["lam"], a["iters"], a["lb"])
                    assert np.array_equal(got[0], a["splits"])
        finally:
            h.close()
    monkeypatch.setenv("NIMBLE_TUNE_PATCH_STRIPS", "1")
    t = fabric(2, 8, "pair")
    h = B.nimble_topo_create(*t.csr(), flags=flags)
    try:
        B.nimble_debug_set_spin_limit(h, 0)
        d = np.floor(np.random.default_rng(9).pareto(1.1, t.n_comm) * 1e6)
        s, l = B.plan(h, d, 0.05, 5)
        assert not B.nimble_debug_patches_gave_up(h)
        ref = oracle.solve(*t.csr(), d, 0.05, 5, flags=flags)
        assert l == ref["lam"] and np.array_equal(s, ref["splits"])
    finally:
        h.close()


@pytest.mark.gpu
def test_a_refused_launch_falls_back(monkeypatch):
    """Where the device does not take the launch of several patches, every kind of solve runs on the
    streaming kernels, once: the next call is on patches again."""
    import oracle
    import torch
    monkeypatch.setenv("NIMBLE_TUNE_PATCH_STRIPS", "3")
    lib = B.load_library()
    t = fabric(7, 6, "pair")
    d = np.floor(np.random.default_rng(9).pareto(1.1, (3, t.n_comm)) * 1e6)
    ref = [oracle.solve(*t.csr(), d[b], 0.05, 30) for b in range(3)]
    warm = oracle.solve(*t.csr(), d[1], 0.05, 9, len0=np.ones(t.n_links))
    a = oracle.solve_adaptive(*t.csr(), d[2], 0.1, 30, 4)
    h = B.nimble_topo_create(*t.csr())
    try:
        for refuse in (True, False):
            for plans in (0, slice(0, 3)):
                if refuse:
                    lib.nimble_debug_refuse_cooperative()
                splits, lam = B.plan(h, d[plans], 0.05, 30)
                assert h.regime == (B.NIMBLE_REGIME_STREAM if refuse else B.NIMBLE_REGIME_PERSISTENT)
                for b in range(3 if plans else 1):
                    got = (splits[b], lam[b]) if plans else (splits, lam)
                    assert got[1] == ref[b]["lam"] and np.array_equal(got[0], ref[b]["splits"]), b
            if refuse:
                lib.nimble_debug_refuse_cooperative()
            ln = torch.ones(t.n_links, dtype=torch.float64, device="cuda:0")
            splits = torch.empty(t.n_paths, dtype=torch.float64, device="cuda:0")
            lam = torch.empty(1, dtype=torch.float64, device="cuda:0")
            B.nimble_plan_solve_warm(h, torch.as_tensor(d[1]).to("cuda:0"), 0.05, 9, ln, splits, lam)
            assert float(lam.item()) == warm["lam"]
            assert np.array_equal(ln.cpu().numpy(), warm["len"])
            if refuse:
                lib.nimble_debug_refuse_cooperative()
            got = _adaptive(h, t, d[2], 0.1, 30, 4)
            assert got[1:] == (a["lam"], a["iters"], a["lb"]) and np.array_equal(got[0], a["splits"])
    finally:
        h.close()


@pytest.mark.gpu
@pytest.mark.parametrize("flags", [0, 1])
@pytest.mark.parametrize("strips", [1, 2, 3])
def test_demands_of_any_range_keep_every_load(monkeypatch, strips, flags):
    """Two separate fabrics, the second with demands and capacities 2^120 times the first one's (no
    single grid holds both), and demands whose total over a patch overflows although no link's
    load does.  Scaling by a power of two changes no bit of any quantity, and sums of whole numbers
    below 2^53 units are exact in any order, so the oracle's bits are demanded."""
    import oracle
    monkeypatch.setenv("NIMBLE_TUNE_PATCH_STRIPS", str(strips))
    one = fabric(2, 8, "pair")
    t = islands(2, one)
    rng = np.random.default_rng(21)
    d1 = np.floor(rng.pareto(1.1, one.n_comm) * 1e6)
    t.cap = np.r_[one.cap, one.cap * 2.0 ** 120]
    for name, d in (("apart", np.r_[d1, d1[::-1] * 2.0 ** 120]),
                    ("further", np.r_[d1 * 2.0 ** -900, d1[::-1] * 2.0 ** 120])):
        if name == "further":
            t.cap = np.r_[one.cap * 2.0 ** -900, one.cap * 2.0 ** 120]
        print(f"[patch] {name} strips={strips} flags={flags}", flush=True)
        ref = oracle.solve(*t.csr(), d, 0.05, 60, flags=flags)
        splits, lam, _ = _solve(t, d[None], 0.05, 60, flags)
        assert lam[0] == ref["lam"] and np.array_equal(splits[0], ref["splits"]), name
        if not flags:
            ref = oracle.solve_adaptive(*t.csr(), d, 0.1, 60, 7)
            h = B.nimble_topo_create(*t.csr())
            try:
                got = _adaptive(h, t, d, 0.1, 60, 7)
            finally:
                h.close()
            assert got[1:] == (ref["lam"], ref["iters"], ref["lb"]), name
            assert np.array_equal(got[0], ref["splits"]), name
    # rail links carry 64 pairs: 2^1022 there, 480 pairs together overflow
    t.cap = np.r_[one.cap, one.cap] * 2.0 ** 900
    d = np.full(t.n_comm, 2.0 ** 1016)
    ref = oracle.solve(*t.csr(), d, 0.05, 60, flags=flags)
    assert np.isfinite(ref["lam"])
    splits, lam, _ = _solve(t, d[None], 0.05, 60, flags)
    assert lam[0] == ref["lam"] and np.array_equal(splits[0], ref["splits"])



@pytest.mark.parametrize("where,status", [(1, 2), (2, 2), (3, 0)])
def test_host_memory_running_out_is_a_status(where, status):
    """The builder of the patch layout out of memory in the calling thread (1) or in a worker (2) is
    a status; a worker that cannot be started (3) is done without.  (2: NIMBLE_ERR_ALLOC)"""
    t = fabric(12, 8, "pair")                    # enough commodities for several workers
    out = np.zeros(12, dtype=np.int64)
    lib = B.load_library()
    for fault in (where, 0):
        lib.nimble_debug_fail_patch_build(fault)
        st = lib.nimble_host_patch_check(t.n_links, t.n_comm, B._hp(t.comm_path_ptr), t.n_paths,
                                         B._hp(t.path_link_ptr), B._hp(t.path_links), 4, 0,
                                         B._hp(out))
        assert st == (status if fault else B.NIMBLE_OK)
        if st == B.NIMBLE_OK:
            assert out[0] == 16 and out[1] == 0


@pytest.mark.gpu
@pytest.mark.parametrize("where", [1, 2, 3])
def test_a_topology_survives_a_failed_patch_build(where):
    """The same in nimble_topo_create, which gives back what it had allocated on the device."""
    lib = B.load_library()
    t = fabric(12, 8, "pair")
    held = lib.nimble_debug_live_allocations()
    lib.nimble_debug_fail_patch_build(where)
    try:
        if where == 3:
            B.nimble_topo_create(*t.csr()).close()
        else:
            with pytest.raises(B.NimbleError) as ei:
                B.nimble_topo_create(*t.csr())
            assert ei.value.status == B.NIMBLE_ERR_ALLOC
    finally:
        lib.nimble_debug_fail_patch_build(0)
    assert lib.nimble_debug_live_allocations() == held
    B.nimble_topo_create(*t.csr()).close()


@pytest.mark.gpu
@pytest.mark.parametrize("large,small,strips", [((3, 8, "pair"), (2, 8, "pair"), 1),
                                                ((8, 8, "xor"), (4, 8, "xor"), 2)])
def test_topologies_share_a_kernel_whatever_their_patches_need(monkeypatch, large, small, strips):
    """A topology made after another one, with smaller patches of the same shape (and so the same
    kernel), leaves the first one's solves as they were; with less and with more than 64 KB of
    LDS."""
    import oracle
    monkeypatch.setenv("NIMBLE_TUNE_PATCH_STRIPS", str(strips))
    monkeypatch.setenv("NIMBLE_TUNE_PATCH_LANES", "1")
    handles = []
    try:
        for f in (large, small):
            t = fabric(*f)
            d = np.floor(np.random.default_rng(5).pareto(1.1, t.n_comm) * 1e6)
            handles.append((t, d, B.nimble_topo_create(*t.csr())))
        for t, d, h in handles + handles:
            splits, lam = B.plan(h, d, 0.05, 20)
            ref = oracle.solve(*t.csr(), d, 0.05, 20)
            assert lam == ref["lam"] and np.array_equal(splits, ref["splits"])
    finally:
        for _, _, h in handles:
            h.close()


@pytest.mark.gpu
def test_phases_can_be_timed_after_a_variable_step_in_one_launch():
    """As after a solve of fixed step: a variable-step solve is a solve, whatever kernels it took."""
    import torch
    for t in (fabric(2, 8, "pair"), fabric(7, 6, "pair")):
        d = np.floor(np.random.default_rng(9).pareto(1.1, t.n_comm) * 1e6)
        h = B.nimble_topo_create(*t.csr())
        try:
            with pytest.raises(B.NimbleError):
                B.nimble_debug_run_phase(h, 0, 1, torch.as_tensor(d).to("cuda:0"))
            before = _adaptive(h, t, d, 0.1, 30, 4)
            for phase in (1, 0, 1):
                B.nimble_debug_run_phase(h, phase, 2, torch.as_tensor(d).to("cuda:0"))
            torch.cuda.synchronize()
            after = _adaptive(h, t, d, 0.1, 30, 4)
            assert before[1:] == after[1:] and np.array_equal(before[0], after[0])
        finally:
            h.close()


@pytest.mark.gpu
def test_a_regime_asked_for_runs_its_own_kernels():
    """Patch kernels are what the library picks by itself.  Asked for by name, the resident regime
    runs its kernels, whose thread per link adds in the oracle's order: demands on no grid give the
    oracle's bits in a batch of more plans than compute units."""
    import oracle
    w = W.make_config(1)
    t, n = w.topo, 257
    d = w.traffic * (1.0 + np.random.default_rng(0).random((n, t.n_comm)))
    h = B.nimble_topo_create(*t.csr())
    try:
        B.plan(h, d[0], w.eps, 30)
        assert h.last_patches == 1 and h.regime == B.NIMBLE_REGIME_RESIDENT
        for regime in (B.NIMBLE_REGIME_STREAM, B.NIMBLE_REGIME_PERSISTENT, B.NIMBLE_REGIME_RESIDENT):
            B.nimble_topo_set_regime(h, regime)
            splits, lam = B.plan(h, d[:3] if regime != B.NIMBLE_REGIME_RESIDENT else d, w.eps, 30)
            assert h.last_patches == 0 and h.regime == regime
        for b in (0, 1, 100, n - 1):
            ref = oracle.solve(*t.csr(), d[b], w.eps, 30)
            assert np.array_equal(splits[b], ref["splits"]) and lam[b] == ref["lam"], b
    finally:
        h.close()


def test_sizes_found_without_building_are_the_layouts():
    """Grids of every size on fabrics and random topologies: groups, parts and local links counted
    from the links' users equal those of the layout that is built (check 19)."""
    for t in (fabric(5, 8, "xor"), fabric(9, 8, "pair"), fabric(6, 6, "own"), direct_mesh(40),
              islands(5, fabric(2, 8, "pair")), _random(16, 100, 1500, 20, 4)):
        built = 0
        for strips in range(1, 17):
            s = B.nimble_host_patch_check(t.n_links, t.n_comm, t.comm_path_ptr, t.n_paths,
                                          t.path_link_ptr, t.path_links, strips)
            assert s["failed"] == 0, s
            built += s["patches"] > 0
        assert built >= 10


@pytest.mark.gpu
def test_patches_are_taken_where_they_are_the_faster_way():
    """Irregular topologies whose patches would share every link with all the others (measured: 3.0 ms
    against 1.8 for 200 iterations, 2.5 against 2.0) are streamed; so is one iteration of a fabric
    whose longer plans run on patches; a batch that shares its launches goes by its own figures.
    Same plans either way."""
    import oracle
    for t, iters, batch, patches in ((_random(11, 300, 20000, 8, 5), 20, 1, False),
                                     (_random(13, 64, 30000, 4, 3), 20, 1, False),
                                     (fabric(16, 8, "pair"), 1, 1, False),
                                     (fabric(16, 8, "pair"), 30, 1, True),
                                     (fabric(5, 8, "xor"), 30, 1, True),
                                     (fabric(5, 8, "xor"), 30, 9, True),
                                     (_random(16, 100, 1500, 20, 4), 30, 1, True)):
        d = np.floor(np.random.default_rng(9).pareto(1.1, (batch, t.n_comm)) * 1e6)
        h = B.nimble_topo_create(*t.csr())
        try:
            splits, lam = B.plan(h, d if batch > 1 else d[0], 0.05, iters)
            assert (h.last_patches > 0) == patches, (t.n_comm, iters, batch, h.last_patches)
        finally:
            h.close()
        ref = oracle.solve(*t.csr(), d[0], 0.05, iters)
        got = (splits[0], lam[0]) if batch > 1 else (splits, lam)
        assert got[1] == ref["lam"] and np.array_equal(got[0], ref["splits"])


OTHER_PROCESS = """
import sys
sys.path[:0] = [sys.argv[1], sys.argv[1] + "/tests"]
import numpy as np
import test_patch as T
B, t = T.B, T.fabric(7, 6, "pair")
d = np.floor(np.random.default_rng(9).pareto(1.1, t.n_comm) * 1e6)
h = B.nimble_topo_create(*t.csr())
splits, lam = B.plan(h, d, 0.05, 30)
a = T._adaptive(h, t, d, 0.1, 30, 4)
np.savez(sys.argv[2], splits=splits, lam=lam, patches=h.last_patches, adaptive=a[0], rest=a[1:])
h.close()
"""


@pytest.mark.gpu
def test_two_processes_share_a_gpu(tmp_path):
    """Cooperative launches are to be had by one process at a time: while this one has its patches, a
    second one gets the same plans from whatever kernels it can launch."""
    import oracle
    import os
    import subprocess
    import sys
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    t = fabric(7, 6, "pair")
    d = np.floor(np.random.default_rng(9).pareto(1.1, t.n_comm) * 1e6)
    h = B.nimble_topo_create(*t.csr())
    try:
        B.plan(h, d, 0.05, 30)
        assert h.last_patches > 1
        out = str(tmp_path / "other.npz")
        r = subprocess.run([sys.executable, "-c", OTHER_PROCESS, root, out], capture_output=True,
                           text=True, timeout=100)
        assert r.returncode == 0, r.stderr[-800:]
        other = np.load(out)
        ref = oracle.solve(*t.csr(), d, 0.05, 30)
        assert float(other["lam"]) == ref["lam"] and np.array_equal(other["splits"], ref["splits"])
        a = oracle.solve_adaptive(*t.csr(), d, 0.1, 30, 4)
        assert other["rest"].tolist() == [a["lam"], a["iters"], a["lb"]]
        assert np.array_equal(other["adaptive"], a["splits"])
        print(f"[patch] the other process had {int(other['patches'])} patches", flush=True)
        splits, lam = B.plan(h, d, 0.05, 30)
        assert h.last_patches > 1 and lam == ref["lam"] and np.array_equal(splits, ref["splits"])
    finally:
        h.close()


# (product slots, lanes, slots per lane) there are kernels for
SHAPES = {(1, 1, q) for q in (1, 2, 3, 4, 6, 8)} | {(1, 2, q) for q in (1, 2, 3, 4)} | \
         {(1, 4, 1), (1, 4, 2)} | {(0, 1, q) for q in (1, 2, 4)} | \
         {(0, 2, q) for q in (1, 2, 4)} | {(0, 4, 1), (0, 4, 2)}


def slotted(product, slots, seed=0):
    """Commodities of up to `slots` slots: four paths over one middle link, reached two ways and
    left two ways (product slots), or paths of four links that have nothing in common (plain)."""
    rng = np.random.default_rng(1000 * product + 10 * slots + seed)
    links, lists = 90, []
    for k in range(70):
        mine = []
        for _ in range(slots if k % 3 else 1 + k % slots):
            e = [int(x) for x in rng.permutation(links)]
            if product:
                mine += [[a, e[4], d] for a in e[:2] for d in e[2:4]]
            else:
                mine += [e[4 * i:4 * i + 4] for i in range(4)]
        lists.append(mine if k % 5 or product else mine[:-1])
    return _topology(links, 1e9 * (1 + np.arange(links) % 7), lists)


def _shapes(strips):
    """The shapes that the topologies of `slotted` have on a grid: shape -> (topology, lanes)."""
    found = {}
    for product in (1, 0):
        for slots in range(1, 9):
            t = slotted(product, slots)
            for lanes in (1, 2, 4):
                s = B.nimble_host_patch_check(t.n_links, t.n_comm, t.comm_path_ptr, t.n_paths,
                                              t.path_link_ptr, t.path_links, strips, lanes)
                assert s["failed"] == 0
                if s["patches"] > 0 and (s["patches"] > 1) == (strips > 1):
                    found.setdefault((s["product"], s["lanes"], s["slots_per_lane"]), (t, lanes))
    return found


@pytest.mark.parametrize("strips", [1, 3])
def test_every_shape_has_a_topology(strips):
    assert set(_shapes(strips)) == SHAPES


@pytest.mark.gpu
@pytest.mark.parametrize("strips", [1, 3])
def test_every_shape_matches_the_oracle(monkeypatch, strips):
    """All kernels: every shape, for one patch and for several, both path costs, fixed and variable
    step."""
    import oracle
    monkeypatch.setenv("NIMBLE_TUNE_PATCH_STRIPS", str(strips))
    for shape, (t, lanes) in sorted(_shapes(strips).items()):
        monkeypatch.setenv("NIMBLE_TUNE_PATCH_LANES", str(lanes))
        d = np.floor(np.random.default_rng(3).pareto(1.1, t.n_comm) * 1e6)
        for flags in (0, 1):
            print(f"[patch] shape {shape} strips={strips} flags={flags}", flush=True)
            h = B.nimble_topo_create(*t.csr(), flags=flags)
            try:
                splits, lam = B.plan(h, d, 0.05, 60)
                assert (h.last_patches > 1) == (strips > 1) and h.last_patches > 0
                ref = oracle.solve(*t.csr(), d, 0.05, 60, flags=flags)
                assert lam == ref["lam"] and np.array_equal(splits, ref["splits"]), shape
                if not flags:
                    got = _adaptive(h, t, d, 0.1, 60, 7)
                    assert h.last_patches > 0
                    ref = oracle.solve_adaptive(*t.csr(), d, 0.1, 60, 7)
                    assert got[1:] == (ref["lam"], ref["iters"], ref["lb"]), shape
                    assert np.array_equal(got[0], ref["splits"]), shape
            finally:
                h.close()


@pytest.mark.gpu
@pytest.mark.parametrize("flags", [0, 1])
@pytest.mark.parametrize("iters", [1, 4, 7])
def test_teams_that_solve_several_plans(monkeypatch, iters, flags):
    """More than twice as many plans as teams, and no multiple of it: what a team counts over its
    exchanges and meetings goes on from plan to plan, for odd and even numbers of exchanges; plans
    without traffic in the middle."""
    import oracle
    monkeypatch.setenv("NIMBLE_TUNE_PATCH_STRIPS", "4")
    for t in (fabric(5, 8, "xor"), fabric(7, 6, "pair")):
        h = B.nimble_topo_create(*t.csr(), flags=flags)
        try:
            B.plan(h, np.ones(t.n_comm), 0.05, 1)
            n = 2 * (256 // h.last_patches) + 3
            d = np.floor(np.random.default_rng(4).pareto(1.1, (n, t.n_comm)) * 1e6)
            d[n // 2] = 0.0
            d[5] = 0.0
            print(f"[patch] {n} plans, {h.last_patches} patches, {iters} iterations", flush=True)
            splits, lam = B.plan(h, d, 0.05, iters)
            assert h.last_patches > 1
            for b in range(n):
                ref = oracle.solve(*t.csr(), d[b], 0.05, iters, flags=flags)
                assert lam[b] == ref["lam"] and np.array_equal(splits[b], ref["splits"]), b
        finally:
            h.close()


@pytest.mark.gpu
@pytest.mark.parametrize("strips,patches", [(2, 4), (3, 9), (5, 25), (6, 36)])
def test_teams_of_one_xcd_and_of_several(monkeypatch, strips, patches):
    """Patches that fit the compute units of one XCD (32) exchange their loads inside it, one team per
    XCD or several; 36 do not.  One plan, as many as fill some XCDs, and more than there are teams."""
    import oracle
    monkeypatch.setenv("NIMBLE_TUNE_PATCH_STRIPS", str(strips))
    t = fabric(6, 6, "pair")
    h = B.nimble_topo_create(*t.csr())
    try:
        d = np.floor(np.random.default_rng(6).pareto(1.1, (70, t.n_comm)) * 1e6)
        ref = [oracle.solve(*t.csr(), x, 0.05, 9) for x in d]
        for n in (1, 11, 70):
            splits, lam = B.plan(h, d[:n], 0.05, 9)
            assert h.last_patches == patches
            assert not B.nimble_debug_patches_gave_up(h)
            for b in range(n):
                assert np.atleast_1d(lam)[b] == ref[b]["lam"], (n, b)
                assert np.array_equal(splits.reshape(n, -1)[b], ref[b]["splits"]), (n, b)
    finally:
        h.close()


def part_of(t, seed, pairs, paths):
    """A fabric of which a share `pairs` of the commodities is planned for, with a share `paths` of their
    candidates (at least one)."""
    rng = np.random.default_rng(seed)
    comm = np.repeat(np.arange(t.n_comm), np.diff(t.comm_path_ptr))
    on = rng.random(t.n_comm) < pairs
    keep = rng.random(t.n_paths) < paths
    some = np.zeros(t.n_comm, dtype=bool)
    some[comm[keep]] = True
    keep[t.comm_path_ptr[:-1][~some]] = True
    keep &= on[comm]
    lens = np.diff(t.path_link_ptr)
    k = int(on.sum())
    zeros = np.zeros(k, dtype=np.int32)
    return W.Topology(n_links=t.n_links, cap=t.cap, n_comm=k,
                      comm_path_ptr=np.concatenate([[0], np.cumsum(np.bincount(
                          comm[keep], minlength=t.n_comm)[on])]).astype(np.int32),
                      n_paths=int(keep.sum()),
                      path_link_ptr=np.concatenate([[0], np.cumsum(lens[keep])]).astype(np.int32),
                      path_links=t.path_links[np.repeat(keep, lens)], src=zeros, dst=zeros,
                      meta=dict(kind="part"))


# (the first three: 274 groups in each of 16 x 16 patches, 310 and 292 in each of 15 x 15, more places than
# 16 bits number)
@pytest.mark.parametrize("what", [(64, 8, "own", 0.05, 0.1), (56, 8, "own", 0.05, 0.4),
                                  (48, 8, "pair", 0.05, 0.3), (48, 8, "xor", 0.2, 0.2),
                                  (16, 8, "pair", 1.0, 1.0), (24, 8, "xor", 1.0, 1.0),
                                  (6, 6, "pair", 1.0, 1.0), (9, 5, "own", 0.7, 0.7)])
@pytest.mark.parametrize("cus", [256, 64])
def test_what_is_chosen_can_be_built(what, cus):
    t = part_of(fabric(*what[:3]), 1, *what[3:])
    chosen = B.nimble_host_patch_choice(t.n_links, t.n_comm, t.comm_path_ptr, t.n_paths, t.path_link_ptr,
                                        t.path_links, cus, cus // 32)
    assert all(c["failed"] == 0 and c["patches"] <= cus for c in chosen), chosen
    assert chosen or cus < 256


@pytest.mark.parametrize("patches,plans,near,teams,us", [
    (1, 1, True, 1, 2.0), (1, 257, True, 256, 4.0), (16, 16, True, 16, 2.0), (16, 17, True, 16, 4.0),
    (20, 1, True, 1, 2.0), (20, 8, True, 8, 2.0), (20, 9, False, 9, 3.0), (20, 12, False, 12, 3.0),
    (20, 13, True, 8, 4.0), (20, 16, True, 8, 4.0), (20, 17, False, 12, 6.0), (32, 9, True, 8, 4.0),
    (33, 1, False, 1, 3.0), (33, 8, False, 7, 6.0), (256, 1, False, 1, 3.0), (256, 3, False, 1, 9.0)])
def test_plans_are_rated_as_they_run(patches, plans, near, teams, us):
    """Teams within one XCD (2 us an iteration) while that takes no more rounds than teams that are spread
    (3 us): the layout is chosen by the microseconds of the teams that the launch then makes."""
    assert B.nimble_host_patch_teams(patches, plans, 2.0, 3.0) == (near, teams, us)


@pytest.mark.gpu
def test_a_stream_under_capture_takes_one_patch():
    """Of a fabric with a layout of one patch and a faster one of several (4 nodes, a NIC per GPU
    reachable from two), an eager plan takes the several, a captured one the single patch."""
    import oracle
    import torch
    t = fabric(4, 8, "xor")
    d = [np.floor(np.random.default_rng(s).pareto(1.1, t.n_comm) * 1e6) for s in (1, 2)]
    ref = [oracle.solve(*t.csr(), x, 0.05, 60) for x in d]
    h = B.nimble_topo_create(*t.csr())
    try:
        dd = [torch.as_tensor(x).to("cuda:0") for x in d]
        out = [(torch.empty(t.n_paths, dtype=torch.float64, device="cuda:0"),
                torch.empty(1, dtype=torch.float64, device="cuda:0")) for _ in d]
        side = torch.cuda.Stream()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.stream(side):
            B.nimble_plan_solve(h, dd[0], 0.05, 60, *out[0])
            torch.cuda.synchronize()
            assert h.last_patches > 1
            with torch.cuda.graph(graph, stream=side):
                B.nimble_plan_solve(h, dd[0], 0.05, 60, *out[0])
            assert h.last_patches == 1
        for _ in range(3):
            out[0][0].zero_()
            B.nimble_plan_solve(h, dd[1], 0.05, 60, *out[1])
            assert h.last_patches > 1
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            for (splits, lam), r in zip(out, ref):
                assert float(lam.item()) == r["lam"]
                assert np.array_equal(splits.cpu().numpy(), r["splits"])
    finally:
        h.close()


@pytest.mark.gpu
def test_a_variable_step_has_a_layout_of_its_own():
    """A fabric whose fixed-step plans run on one patch that has no room for the weights of a variable
    step: that one is solved on several."""
    import oracle
    t = fabric(5, 6, "xor")
    d = np.floor(np.random.default_rng(1).pareto(1.1, t.n_comm) * 1e6)
    h = B.nimble_topo_create(*t.csr())
    try:
        splits, lam = B.plan(h, d, 0.05, 60)
        assert h.last_patches == 1
        ref = oracle.solve(*t.csr(), d, 0.05, 60)
        assert lam == ref["lam"] and np.array_equal(splits, ref["splits"])
        got = _adaptive(h, t, d, 0.1, 60, 7)
        assert h.last_patches > 1
        ref = oracle.solve_adaptive(*t.csr(), d, 0.1, 60, 7)
        assert got[1:] == (ref["lam"], ref["iters"], ref["lb"])
        assert np.array_equal(got[0], ref["splits"])
    finally:
        h.close()


@pytest.mark.gpu
@pytest.mark.parametrize("every", [1, 7])
@pytest.mark.parametrize("strips", [6, 7, 9, 14])
def test_a_variable_step_between_xcds_with_lists_of_any_length(monkeypatch, strips, every):
    """Teams of more than 32 patches meet through a leader per XCD: 36, 49, 81 and 196 patches, so that the
    eight leaders have 4 and 5, 6 and 7, 10 and 11, 24 and 25 of them."""
    import oracle
    monkeypatch.setenv("NIMBLE_TUNE_PATCH_STRIPS", str(strips))
    t = fabric(7, 6, "pair")
    d = np.floor(np.random.default_rng(strips).pareto(1.1, t.n_comm) * 1e6)
    print(f"[patch adaptive] {strips} x {strips} patches, a check every {every}", flush=True)
    h = B.nimble_topo_create(*t.csr())
    try:
        for iters in (1, 41):
            got = _adaptive(h, t, d, 0.1, iters, every)
            assert h.last_patches == strips * strips
            ref = oracle.solve_adaptive(*t.csr(), d, 0.1, iters, every)
            assert got[1:] == (ref["lam"], ref["iters"], ref["lb"])
            assert np.array_equal(got[0], ref["splits"])
    finally:
        h.close()


@pytest.mark.gpu
@pytest.mark.parametrize("what,third", [((6, 6, "pair"), True), ((13, 8, "xor"), True),
                                        ((4, 8, "own"), False), ((3, 8, "xor"), False)])
def test_a_third_layout_for_the_variable_step(what, third):
    """Fabrics whose layout for one plan is in blocks, which have no variable step: that one is solved on
    the layout kept for it alone, or on one patch, which needs no other layout."""
    import oracle
    t = fabric(*what)
    chosen = B.nimble_host_patch_choice(t.n_links, t.n_comm, t.comm_path_ptr, t.n_paths, t.path_link_ptr,
                                        t.path_links)
    assert chosen[0]["blocks"] == 1 and chosen[-1]["variable_only"] == third
    d = np.floor(np.random.default_rng(1).pareto(1.1, t.n_comm) * 1e6)
    print(f"[patch adaptive] third layout of {what}", flush=True)
    h = B.nimble_topo_create(*t.csr())
    try:
        splits, lam = B.plan(h, d, 0.05, 300)
        assert h.last_patches in (c["patches"] for c in chosen)
        ref = oracle.solve(*t.csr(), d, 0.05, 300)
        assert lam == ref["lam"] and np.array_equal(splits, ref["splits"])
        got = _adaptive(h, t, d, 0.1, 60, 7)
        assert h.last_patches == (chosen[-1]["patches"] if third else 1)
        ref = oracle.solve_adaptive(*t.csr(), d, 0.1, 60, 7)
        assert got[1:] == (ref["lam"], ref["iters"], ref["lb"])
        assert np.array_equal(got[0], ref["splits"])
    finally:
        h.close()


@pytest.mark.gpu
@pytest.mark.parametrize("blocks", [0, 1])
@pytest.mark.parametrize("grid,patches", [("2", 4), ("4x5", 20), ("6", 36), ("14", 196)])
def test_fractional_loads_of_every_link(monkeypatch, grid, patches, blocks):
    """One iteration from unit lengths on demands that lie on no common grid: choices do not depend on
    loads yet, so the length of every link shows its load.  The oracle adds up to K demands one after the
    other and the patches round each part twice and add up to 31: with the width rounded alike and u =
    2^-53, length - 1 = eps * load / cap / rho differs by at most 2 (K + 31 + 8) u relative, and the
    length itself by a rounding, 2 u."""
    import oracle
    import torch
    monkeypatch.setenv("NIMBLE_TUNE_PATCH_STRIPS", grid)
    monkeypatch.setenv("NIMBLE_TUNE_PATCH_BLOCKS", str(blocks))
    t = fabric(7, 6, "pair")
    rng = np.random.default_rng(12)
    print(f"[patch] fractional loads, grid {grid}, blocks {blocks}", flush=True)
    h = B.nimble_topo_create(*t.csr())
    try:
        for _ in range(3):
            d = rng.pareto(1.1, t.n_comm) * 1e6 * (1.0 + rng.random(t.n_comm))
            length = torch.ones(t.n_links, dtype=torch.float64, device="cuda:0")
            splits = torch.empty(t.n_paths, dtype=torch.float64, device="cuda:0")
            lam = torch.empty(1, dtype=torch.float64, device="cuda:0")
            B.nimble_plan_solve_warm(h, torch.as_tensor(d).to("cuda:0"), 0.5, 1, length, splits, lam)
            assert h.last_patches == patches and not B.nimble_debug_patches_gave_up(h)
            ref = oracle.solve(*t.csr(), d, 0.5, 1, len0=np.ones(t.n_links))
            u, rel = 2.0 ** -53, 2.0 * (t.n_comm + 39) * 2.0 ** -53
            assert np.array_equal(splits.cpu().numpy(), ref["splits"])
            assert np.all(np.abs(length.cpu().numpy() - ref["len"]) <= rel * (ref["len"] - 1.0) + 2 * u)
            assert (ref["len"] > 1.0).mean() > 0.5
            assert abs(float(lam.item()) - ref["lam"]) <= rel * ref["lam"]
    finally:
        h.close()
