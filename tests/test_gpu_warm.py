"""GPU parity of nimble_plan_solve_warm against the oracle's warm start, through the C ABI."""
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


def gpu_warm(B, h, topo, demand, eps, iters, len0):
    import torch
    d = torch.as_tensor(np.ascontiguousarray(demand, dtype=np.float64)).to("cuda:0")
    ln = torch.as_tensor(np.ascontiguousarray(len0, dtype=np.float64)).to("cuda:0")
    splits = torch.full((topo.n_paths,), float("nan"), dtype=torch.float64, device="cuda:0")
    lam = torch.full((1,), float("nan"), dtype=torch.float64, device="cuda:0")
    B.nimble_plan_solve_warm(h, d, eps, iters, ln, splits, lam)
    torch.cuda.synchronize()
    return splits.cpu().numpy(), float(lam.item()), ln.cpu().numpy()


@pytest.mark.parametrize("patches", [True, False])
@pytest.mark.parametrize("cfg,t1,t2,flags", [(0, 40, 60, 0), (1, 50, 70, 0), (1, 50, 70, 1),
                                             (3, 30, 40, 0), (4, 12, 13, 0)])
def test_two_solves_in_a_row_match_the_oracle(oracle_mod, B, monkeypatch, cfg, t1, t2, flags,
                                              patches):
    """A first plan from unit lengths, then a plan for different traffic from the lengths the
    first one returned: splits, lambda and the returned lengths are bit-identical to the
    oracle, on the patch kernels and, without them, streamed on the fused (config 3) and the tiled
    (config 4) reduce alike."""
    if not patches:
        monkeypatch.setenv("NIMBLE_TUNE_PATCH_STRIPS", "0")
    w = W.make_config(cfg)
    t = w.topo
    print(f"[warm] config {cfg}", flush=True)
    d2 = np.roll(w.traffic, 7)
    h = B.nimble_topo_create(t.n_links, t.cap, t.n_comm, t.comm_path_ptr, t.n_paths,
                             t.path_link_ptr, t.path_links, flags)
    try:
        s1, l1, len1 = gpu_warm(B, h, t, w.traffic, w.eps, t1, np.ones(t.n_links))
        s2, l2, len2 = gpu_warm(B, h, t, d2, w.eps, t2, len1)
        assert h.regime == B.NIMBLE_REGIME_STREAM
        assert (h.last_patches > 0) == patches
    finally:
        h.close()
    r1 = oracle_mod.solve(*t.csr(), w.traffic, w.eps, t1, flags=flags, len0=np.ones(t.n_links))
    assert np.array_equal(s1, r1["splits"]) and l1 == r1["lam"]
    assert np.array_equal(len1, r1["len"])
    r2 = oracle_mod.solve(*t.csr(), d2, w.eps, t2, flags=flags, len0=r1["len"])
    assert np.array_equal(s2, r2["splits"]) and l2 == r2["lam"]
    assert np.array_equal(len2, r2["len"])


def test_continuation_equals_one_long_solve(B):
    """Property that holds at any size: 400 + 600 warm iterations on the 64-node fabric make
    the choices of one cold solve of 1000 iterations."""
    w = W.make_config(4)
    t = w.topo
    h = B.nimble_topo_create(*t.csr())
    try:
        full, lam_full = B.plan(h, w.traffic, w.eps, 1000)
        s1, _, len1 = gpu_warm(B, h, t, w.traffic, w.eps, 400, np.ones(t.n_links))
        s2, _, _ = gpu_warm(B, h, t, w.traffic, w.eps, 600, len1)
    finally:
        h.close()
    counts = np.rint(s1 * 400) + np.rint(s2 * 600)
    assert np.array_equal(counts, np.rint(full * 1000))


def test_null_length_pointer_is_refused(B):
    import torch
    w = W.make_config(0)
    h = B.nimble_topo_create(*w.topo.csr())
    d = torch.zeros(w.topo.n_comm, dtype=torch.float64, device="cuda:0")
    sp = torch.zeros(w.topo.n_paths, dtype=torch.float64, device="cuda:0")
    lam = torch.zeros(1, dtype=torch.float64, device="cuda:0")
    try:
        st = B.load_library().nimble_plan_solve_warm(h.handle, d.data_ptr(), 0.1, 10, None,
                                                     sp.data_ptr(), lam.data_ptr(), None)
        assert st == B.NIMBLE_ERR_INVALID
    finally:
        h.close()
