"""GPU invariants of the library that need no oracle: collision fixed points,
conservation, poisoned destination buffers, checkpoint/resume, graph versus
direct launches, streams, device-pointer I/O, the FP64 reductions and the
error paths of the ABI."""
import numpy as np
import pytest
import torch

from gpu_common import rel_u, run_gpu, run_oracle
from paper_2002_02503_amd import lbm

pytestmark = pytest.mark.gpu


def _fields(dims, seed=0, amp=0.05):
    rng = np.random.default_rng(seed)
    nx, ny, nz = dims
    u = rng.uniform(-amp, amp, size=(3, nz, ny, nx))
    rho = 1.0 + rng.uniform(-0.01, 0.01, size=(nz, ny, nx))
    return rho, u


@pytest.mark.parametrize("dtype", ["fp64", "fp32"])
@pytest.mark.parametrize("lattice", ["D3Q19", "D3Q39"])
def test_uniform_flow_stays_uniform(lattice, dtype):
    dims = (64, 4, 3)
    U = np.array([0.08, -0.05, 0.03])
    rho = np.full((3, 4, 64), 1.02)
    u = np.broadcast_to(U.reshape(3, 1, 1, 1), (3, 3, 4, 64)).copy()
    r, uu = run_gpu(lattice, dims, 0.6, dtype, rho, u, 50)
    tol = 1e-14 if dtype == "fp64" else 1e-7
    assert np.abs(uu - u).max() < tol
    assert np.abs(r - rho).max() < tol
    # every site identical, bit for bit
    assert np.all(uu == uu[:, :1, :1, :1])


def test_poisoned_buffers_are_fully_overwritten():
    """Both population buffers filled with NaN bytes before init: every site
    of every step's destination is written, so nothing non-finite appears,
    and the result equals a run on clean buffers bit for bit."""
    dims = (100, 7, 6)
    rho, u = _fields(dims, 1)
    clean = run_gpu("D3Q19", dims, 0.6, "fp32", rho, u, 7)
    with lbm.Simulation("D3Q19", dims, 0.6, dtype="fp32") as sim:
        for b in sim._bufs:
            b.fill_(0xFF)
        sim.init(rho, u).step(7)
        r, uu = sim.moments()
    assert np.isfinite(r).all() and np.isfinite(uu).all()
    assert np.array_equal(r, clean[0]) and np.array_equal(uu, clean[1])


@pytest.mark.parametrize("dtype", ["fp32", "fp16", "bf16", "fp64"])
def test_checkpoint_resume_is_bitwise(dtype):
    dims = (48, 10, 9)
    rho, u = _fields(dims, 2)
    with lbm.Simulation("D3Q19", dims, 0.58, dtype=dtype) as a:
        a.init(rho, u).step(13)
        ck = a.get_state()
        a.step(17)
        ra, ua = a.moments()
        assert a.t == 30
    with lbm.Simulation("D3Q19", dims, 0.58, dtype=dtype) as b:
        b.set_state(ck)
        assert b.t == 13
        b.step(17)
        rb, ub = b.moments()
    assert np.array_equal(ra, rb) and np.array_equal(ua, ub)


def test_checkpoint_rejects_other_geometry():
    rho, u = _fields((16, 8, 8), 3)
    with lbm.Simulation("D3Q19", (16, 8, 8), 0.6) as a:
        ck = a.init(rho, u).get_state()
    with lbm.Simulation("D3Q19", (8, 16, 8), 0.6) as b:
        with pytest.raises(lbm.LBMError) as e:
            b.set_state(ck)
        assert e.value.name == "LBM_EINVAL"


@pytest.mark.parametrize("chunk", [1, 2, 7, 16])
def test_graph_launches_equal_direct_launches(chunk):
    """Steps issued as captured graphs (chunks of `chunk` steps plus a
    remainder) compute the same bits as one launch per step; repeated graph
    replays with host work between them stay identical."""
    dims = (80, 9, 7)
    rho, u = _fields(dims, 4)
    ref = run_gpu("D3Q19", dims, 0.6, "fp32", rho, u, 40, graph_chunk=1)
    with lbm.Simulation("D3Q19", dims, 0.6, dtype="fp32", graph_chunk=chunk) as sim:
        sim.init(rho, u).prepare()
        for n in [5, 20, 15]:
            sim.step(n)
            sim.sync()
            _ = np.sum(np.arange(1000))  # host work between replays
        r, uu = sim.moments()
    assert np.array_equal(r, ref[0]) and np.array_equal(uu, ref[1])


def test_runs_on_a_caller_stream():
    dims = (64, 8, 8)
    rho, u = _fields(dims, 5)
    ref = run_gpu("D3Q19", dims, 0.6, "fp32", rho, u, 20)
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        with lbm.Simulation("D3Q19", dims, 0.6, dtype="fp32", stream=s) as sim:
            sim.init(rho, u).step(20)
            r, uu = sim.moments()
    assert np.array_equal(r, ref[0]) and np.array_equal(uu, ref[1])


def test_device_pointer_io_matches_host_io():
    dims = (40, 6, 5)
    rho, u = _fields(dims, 6)
    ref = run_gpu("D3Q19", dims, 0.6, "fp32", rho, u, 9)
    with lbm.Simulation("D3Q19", dims, 0.6, dtype="fp32") as sim:
        sim.init(torch.from_numpy(rho).cuda(), torch.from_numpy(u).cuda()).step(9)
        r, uu = sim.moments(device=True)
    assert np.array_equal(r.cpu().numpy(), ref[0]) and np.array_equal(uu.cpu().numpy(), ref[1])


def test_totals_and_residual_match_numpy():
    dims = (50, 11, 7)
    rho, u = _fields(dims, 7)
    r_ref, u_ref = run_oracle("D3Q19", dims, 0.6, rho, u, 12)
    with lbm.Simulation("D3Q19", dims, 0.6, dtype="fp64") as sim:
        sim.init(rho, u)
        t0 = sim.totals()[0]
        sim.step(12)
        t1 = sim.totals()[0]
        r, uu = sim.moments()
        res = sim.residual(r_ref, u_ref)
    assert abs(t1[0] - np.sum(r)) < 1e-10
    assert np.abs(t1[1:] - np.sum(r * uu, axis=(1, 2, 3))).max() < 1e-12
    assert abs(t1[0] - t0[0]) / t0[0] < 1e-14
    assert np.abs(t1[1:] - t0[1:]).max() / t0[0] < 1e-14
    du = uu - u_ref
    assert abs(res["u_max"] - np.abs(du).max()) <= 1e-18 + 1e-12 * np.abs(du).max()
    assert abs(res["u_l2"] - np.sqrt(np.sum(du * du))) <= 1e-12 * np.sqrt(np.sum(du * du)) + 1e-18
    dr = r - r_ref
    assert abs(res["rho_max"] - np.abs(dr).max()) <= 1e-18 + 1e-12 * np.abs(dr).max()


def test_error_paths():
    dims = (16, 8, 8)
    rho, u = _fields(dims, 8)
    with lbm.Simulation("D3Q19", dims, 0.6) as sim:
        with pytest.raises(lbm.LBMError) as e:
            sim.step(1)
        assert e.value.name == "LBM_ESTATE"
        with pytest.raises(lbm.LBMError) as e:
            sim.moments()
        assert e.value.name == "LBM_ESTATE"
        for K in [1, 4]:
            with pytest.raises(lbm.LBMError) as e:
                lbm._check(sim.lib.lbm_set_hermite_order(sim.h, K))
            assert e.value.name == "LBM_EINVAL"
        sim.init(rho, u)
        with pytest.raises(lbm.LBMError) as e:
            lbm._check(sim.lib.lbm_set_hermite_order(sim.h, 2))
        assert e.value.name == "LBM_ESTATE"
        with pytest.raises(lbm.LBMError) as e:
            sim.step(-1)
        assert e.value.name == "LBM_EINVAL"
        with pytest.raises(lbm.LBMError) as e:
            lbm._check(sim.lib.lbm_set_launch(sim.h, 96, 0))
        assert e.value.name == "LBM_EINVAL"


def test_non_finite_state_is_reported():
    """A checkpoint whose populations are NaN restores fine, and lbm_totals
    then reports LBM_ENUMERIC (the check is on the host, the kernels simply
    propagate the NaN)."""
    dims = (16, 8, 8)
    rho, u = _fields(dims, 9)
    with lbm.Simulation("D3Q19", dims, 0.6, dtype="fp32") as sim:
        ck = sim.init(rho, u).get_state()
        payload = ck[64:].view(np.float32)
        payload[:] = np.nan
        sim.set_state(ck)
        with pytest.raises(lbm.LBMError) as e:
            sim.totals()
        assert e.value.name == "LBM_ENUMERIC"


def test_batch_of_equal_boxes_equals_single_boxes():
    """Two identical boxes in one batch each evolve exactly like the single box."""
    dims = (24, 20, 18)
    rho, u = _fields(dims, 10)
    single = run_gpu("D3Q19", dims, 0.65, "fp32", rho, u, 30)
    with lbm.Simulation("D3Q19", [dims, dims], [0.65, 0.65], dtype="fp32") as sim:
        sim.init(np.concatenate([rho.ravel()] * 2), np.concatenate([u.reshape(3, -1)] * 2, axis=1))
        sim.step(30)
        r, uu = sim.moments()
    for k, ub in enumerate(sim.split_boxes(uu)):
        assert np.abs(ub - single[1]).max() < 1e-7, k


@pytest.mark.parametrize("lattice,dims,dtype", [("D3Q19", (64, 12, 10), "fp32"), ("D3Q19", (64, 12, 10), "bf16"),
                                                ("D3Q39", (48, 9, 7), "fp32"), ("D3Q39", (150, 6, 4), "fp32")])
def test_tuning_restores_state_and_keeps_results(lattice, dims, dtype, tmp_path):
    """lbm_tune times every candidate launch on the live state, restores it,
    and whatever it picks computes the same bits; its cache is reused."""
    rho, u = _fields(dims, 11)
    ref = run_gpu(lattice, dims, 0.6, dtype, rho, u, 30)
    cache = str(tmp_path / "tune.txt")
    with lbm.Simulation(lattice, dims, 0.6, dtype=dtype) as sim:
        sim.init(rho, u).step(10)
        sim.tune(steps=5, cache=cache)
        assert sim.t == 10
        chosen = sim.info()
        sim.step(20)
        r, uu = sim.moments()
    assert np.array_equal(r, ref[0]) and np.array_equal(uu, ref[1])
    lines = open(cache).read().splitlines()
    assert len(lines) == 1
    with lbm.Simulation(lattice, dims, 0.6, dtype=dtype) as sim2:
        sim2.init(rho, u).tune(steps=5, cache=cache)
        info = sim2.info()
        assert (info["kernel"], info["block"]) == (chosen["kernel"], chosen["block"])
    assert len(open(cache).read().splitlines()) == 1


def test_tuning_a_batch_keeps_results(tmp_path):
    dims = [(20, 17, 9), (33, 8, 12), (16, 16, 16)]
    rng = np.random.default_rng(12)
    n = sum(a * b * c for a, b, c in dims)
    rho = 1 + rng.uniform(-0.01, 0.01, n)
    u = rng.uniform(-0.05, 0.05, (3, n))
    with lbm.Simulation("D3Q19", dims, [0.6, 0.7, 0.8], dtype="fp32") as a:
        a.init(rho, u).step(25)
        ra, ua = a.moments()
    with lbm.Simulation("D3Q19", dims, [0.6, 0.7, 0.8], dtype="fp32") as b:
        b.init(rho, u).tune(steps=4, cache=str(tmp_path / "c.txt")).step(25)
        rb, ub = b.moments()
        assert b.info()["block"] in (64, 128, 256)
    assert np.array_equal(ra, rb) and np.array_equal(ua, ub)


def test_tuning_cache_with_bad_entries(tmp_path):
    """A cache line edited to values the library cannot launch (unknown kernel,
    a block that is not a multiple of 64, a negative grid) is replaced by valid
    ones, and the run still computes the reference bits."""
    dims = (96, 6, 5)
    rho, u = _fields(dims, 13)
    ref = run_gpu("D3Q19", dims, 0.6, "fp32", rho, u, 12)
    cache = tmp_path / "tune.txt"
    with lbm.Simulation("D3Q19", dims, 0.6, dtype="fp32") as sim:
        sim.init(rho, u).tune(steps=3, cache=str(cache))
    key = open(cache).read().splitlines()[-1].split(" | ")[0]
    with open(cache, "a") as f:
        f.write(key + " | 99 96 -5\n")
        f.write("garbage without a separator\n")
    with lbm.Simulation("D3Q19", dims, 0.6, dtype="fp32") as sim:
        sim.init(rho, u).tune(steps=3, cache=str(cache))
        info = sim.info()
        assert info["block"] in (64, 128, 192, 256) and info["grid"] >= 0
        sim.step(12)
        r, uu = sim.moments()
    assert np.array_equal(r, ref[0]) and np.array_equal(uu, ref[1])


def test_tuning_cache_of_another_candidate_set(tmp_path):
    """An entry without the mark of this library's candidates (an older file) is
    not taken: the call times them and appends its own choice."""
    rho, u = _fields((24, 20, 9), 14)
    cache = tmp_path / "tune.txt"
    with lbm.Simulation("D3Q19", (24, 20, 9), 0.6, dtype="fp32") as sim:
        sim.init(rho, u).tune(steps=2, cache=str(cache))
    key = open(cache).read().splitlines()[-1].split(" | ")[0]
    old = key[:key.index(" geometry=") + len(" geometry=") + 16]
    cache.write_text(old + f" | {lbm.KERNELS['scalar']} 64 0\n")
    with lbm.Simulation("D3Q19", (24, 20, 9), 0.6, dtype="fp32") as sim:
        sim.init(rho, u).tune(steps=2, cache=str(cache))
        sim.tune(steps=2, cache=str(cache))
    lines = open(cache).read().splitlines()
    assert len(lines) == 2 and lines[1].startswith(key + " | ")


@pytest.mark.parametrize("K", [2, 3])
def test_fp32_rounding_errors_of_the_momentum_do_not_add_up(K):
    """The mean of the momentum (and density) after 100 steps in FP32 against
    the same run in FP64.  A site's populations, of size G ~ W u / T0 <= 2 in
    stored units, are rounded to half a unit in the last place of 1 .. 2, on
    average 2^-23 / sqrt(12), so an unbiased error of the momentum is about
    sqrt(6) 2^-23 / sqrt(12) / 36 a site and step (six populations carry each
    component, stored in units of 1/36) and 1/sqrt(sites) of it in the mean; the
    bound is four times its sum over the steps.  A bias would grow with the
    steps instead of their root."""
    nx, ny, steps = 96, 64, 100
    unbiased = np.sqrt(6 / 12) * 2.0**-23 / 36 * np.sqrt(steps / (nx * ny))
    y, x = np.meshgrid(np.arange(ny) * 2 * np.pi / ny, np.arange(nx) * 2 * np.pi / nx, indexing="ij")
    rho = (1 + 0.005 * np.cos(x + 2 * y))[None]
    drift = []
    for tau in (0.51, 0.6, 0.8, 1.0):
        for seed, flow in ((1, 0.0), (2, 0.1), (3, 0.02), (4, 0.05), (5, 0.07), (6, 0.0)):
            rng = np.random.default_rng(seed)
            d = rng.normal(size=2)
            u = np.stack([0.03 * np.sin(y * rng.integers(0, 3) + x * rng.integers(1, 4) + rng.uniform(0, 6))
                          for _ in range(2)]) + flow * (d / np.linalg.norm(d))[:, None, None]
            mean = {}
            for dtype in ("fp64", "fp32"):
                with lbm.Simulation("D2Q9", (nx, ny, 1), tau, dtype=dtype, K=K) as sim:
                    mean[dtype] = sim.init(rho, u[:, None]).step(steps).totals()[0, :3] / (nx * ny)
            drift.append(np.abs(mean["fp32"] - mean["fp64"]).max())
    assert np.mean(drift) <= 4 * unbiased, (np.mean(drift), unbiased)
