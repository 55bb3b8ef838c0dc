"""The tile kernel (k_step_tile: several time steps per launch in LDS) and the
library's own choice of kernel against the one-site step: the same bits at the
edges of the plans (partial tiles, whole x-rows and pieces of them, sides of
one to three sites, rings wider than a tile), for every storage type and
collision kind, step counts that leave a shorter last launch, and captured
graphs replayed around eager work."""
import numpy as np
import pytest

from gpu_common import run_gpu

pytestmark = pytest.mark.gpu


def _fields(lattice, dims, seed):
    rng = np.random.default_rng(seed)
    nx, ny, nz = dims
    D = 2 if lattice == "D2Q9" else 3
    return 1.0 + rng.uniform(-0.01, 0.01, size=(nz, ny, nx)), rng.uniform(-0.05, 0.05, size=(D, nz, ny, nx))


CASES = [
    ("D2Q9", (64, 64, 1), "fp64", {}),            # 8 x 4 tiles, 8 steps
    ("D2Q9", (65, 33, 1), "fp32", {}),            # partial tiles in x and y
    ("D2Q9", (5, 9, 1), "fp32", {"K": 2}),        # whole rows; the ring wraps
    ("D2Q9", (1, 9, 1), "fp32", {}),
    ("D2Q9", (9, 1, 1), "fp64", {}),
    ("D2Q9", (2, 2, 1), "fp16", {}),
    ("D2Q9", (3, 3, 1), "fp32", {}),              # fewer steps: ring of at most 3
    ("D2Q9", (601, 400, 1), "bf16", {}),          # 32 x 16 tiles, 5 steps
    ("D2Q9", (300, 200, 1), "fp32", {"collision": "bgk"}),
    ("D3Q19", (16, 16, 16), "fp32", {}),          # whole rows, 3 steps
    ("D3Q19", (32, 32, 32), "fp16", {"theta": 0.5}),
    ("D3Q19", (32, 32, 32), "fp64", {"theta": 0.5}),
    ("D3Q19", (17, 5, 3), "fp64", {}),
    ("D3Q19", (1, 1, 7), "fp32", {}),
    ("D3Q19", (2, 3, 2), "bf16", {}),
    ("D3Q19", (64, 24, 7), "fp32", {}),
    ("D3Q15", (40, 30, 23), "fp32", {"collision": "bgk"}),
    ("D3Q15", (24, 40, 32), "fp64", {"K": 2}),
]


@pytest.mark.parametrize("lattice,dims,dtype,kw", CASES)
@pytest.mark.parametrize("steps", [1, 2, 23])
def test_tile_equals_one_site_step(lattice, dims, dtype, kw, steps):
    rho, u = _fields(lattice, dims, seed=steps + sum(dims))
    a = run_gpu(lattice, dims, 0.6, dtype, rho, u, steps, kernel="tile", **kw)
    b = run_gpu(lattice, dims, 0.6, dtype, rho, u, steps, kernel="scalar", **kw)
    assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])


@pytest.mark.parametrize("chunk", [1, 3, 8, 20, 32])
def test_tile_graph_chunks(chunk):
    """Chunks shorter than one launch, whole launches and cut ones, replayed
    with reads of the state between the replays."""
    from paper_2002_02503_amd import lbm

    dims = (64, 48, 1)
    rho, u = _fields("D2Q9", dims, seed=chunk)
    with lbm.Simulation("D2Q9", dims, 0.57, dtype="fp32", kernel="tile", graph_chunk=chunk) as a, \
            lbm.Simulation("D2Q9", dims, 0.57, dtype="fp32", kernel="scalar", graph_chunk=1) as b:
        a.init(rho, u)
        b.init(rho, u)
        for n in (77, 40, 1, 64):
            a.step(n)
            b.step(n)
            ra, rb = a.moments(), b.moments()
            assert a.t == b.t and np.array_equal(ra[0], rb[0]) and np.array_equal(ra[1], rb[1])
            assert np.array_equal(a.totals(), b.totals())


def test_tile_refusals_and_the_default_choice():
    from paper_2002_02503_amd import lbm

    def kernel_of(*args, **kw):
        with lbm.Simulation(*args, torch_memory=False, **kw) as sim:
            return sim.info()["kernel"]

    for args in [("D3Q39", (16, 16, 16), 0.6), ("D3Q19", (128, 128, 128), 0.6),
                 ("D3Q19", [(16, 16, 16), (8, 8, 8)], [0.6, 0.7])]:
        with pytest.raises(lbm.LBMError) as e:
            lbm.Simulation(*args, kernel="tile", torch_memory=False)
        assert e.value.name == "LBM_EINVAL"
    names = {v: k for k, v in lbm.KERNELS.items()}
    assert names[kernel_of("D2Q9", (64, 64, 1), 0.8)] == "tile"
    assert names[kernel_of("D3Q19", (32, 32, 32), 0.8)] == "tile"
    assert names[kernel_of("D3Q19", (128, 128, 128), 0.8)] == "two_step"
    # a launch shape is the one-site step's
    assert names[kernel_of("D3Q19", (32, 32, 32), 0.8, block=128)] == "scalar"
    assert names[kernel_of("D3Q39", (32, 32, 32), 0.8)] == "scalar"
    # where the rings cost more than they save
    assert names[kernel_of("D3Q19", (200, 200, 1), 0.8)] == "scalar"
    assert names[kernel_of("D2Q9", (100000, 1, 1), 0.8)] == "scalar"
    assert names[kernel_of("D2Q9", (1024, 1024, 1), 0.8, dtype="fp16")] == "scalar"


def test_default_choice_resumes_and_switches_mid_run():
    """The default (tile) kernel's state is the natural one: a checkpoint goes
    to and from the in-place steps, and a switch continues bit for bit."""
    from paper_2002_02503_amd import lbm

    dims = (33, 20, 11)
    rho, u = _fields("D3Q19", dims, seed=3)
    ref = run_gpu("D3Q19", dims, 0.6, "fp32", rho, u, 24, kernel="scalar")
    with lbm.Simulation("D3Q19", dims, 0.6, dtype="fp32") as sim, \
            lbm.Simulation("D3Q19", dims, 0.6, dtype="fp32", kernel="twist") as other:
        sim.init(rho, u).step(5)
        ck = sim.get_state()
        for kernel, n in [("twist", 3), ("auto", 6), ("in_place", 1), ("tile", 7), ("scalar", 1), ("auto", 1)]:
            assert lbm.STATUS[sim.lib.lbm_set_kernel(sim.h, lbm.KERNELS[kernel])] == "LBM_OK"
            sim.step(n)
        r, uu = sim.moments()
        other.set_state(ck)
        other.step(19)
        r2, u2 = other.moments()
    assert np.array_equal(r, ref[0]) and np.array_equal(uu, ref[1])
    assert np.array_equal(r2, ref[0]) and np.array_equal(u2, ref[1])
