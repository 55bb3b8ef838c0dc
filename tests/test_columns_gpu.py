"""The two-step kernel on columns of any size against the one-site step: the
same bits for pieces of rows with a narrower last one, sides of one to three
sites, narrow last rows of columns, states on both sides of its store policy,
every storage type and collision kind; and the library's choice of it."""
import numpy as np
import pytest

from gpu_common import run_gpu

pytestmark = pytest.mark.gpu


def _fields(dims, seed):
    rng = np.random.default_rng(seed)
    nx, ny, nz = dims
    return 1.0 + rng.uniform(-0.01, 0.01, size=(nz, ny, nx)), rng.uniform(-0.05, 0.05, size=(3, nz, ny, nx))


CASES = [
    ("D3Q19", (201, 15, 7), "fp32", {"theta": 0.5}),   # rows of 101 and 100
    ("D3Q19", (129, 9, 5), "fp64", {}),                # 65 and 64
    ("D3Q19", (257, 23, 3), "fp16", {}),               # 86, 86, 85
    ("D3Q19", (1, 1, 1), "fp32", {}),
    ("D3Q19", (2, 3, 1), "fp64", {"theta": 0.5}),
    ("D3Q19", (3, 2, 2), "bf16", {}),
    ("D3Q19", (8, 169, 12), "fp32", {"K": 2}),         # 57 rows a column, the last 55
    ("D3Q19", (64, 8, 4), "fp32", {}),                 # the aligned tile
    ("D3Q19", (96, 6, 5), "fp32", {"collision": "bgk"}),
    ("D3Q15", (100, 41, 9), "fp64", {}),
    ("D3Q15", (33, 50, 6), "fp32", {"theta": 0.3}),
    ("D3Q19", (100, 100, 60), "fp32", {}),             # 46 MB: cached stores
]


@pytest.mark.parametrize("lattice,dims,dtype,kw", CASES)
@pytest.mark.parametrize("steps", [1, 2, 15])
def test_columns_equal_one_site_step(lattice, dims, dtype, kw, steps):
    rho, u = _fields(dims, seed=steps + sum(dims))
    a = run_gpu(lattice, dims, 0.6, dtype, rho, u, steps, kernel="columns", **kw)
    b = run_gpu(lattice, dims, 0.6, dtype, rho, u, steps, kernel="scalar", **kw)
    assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])


@pytest.mark.parametrize("grid", [1, 5, 16, 999])
def test_columns_any_grid(grid):
    dims = (70, 31, 9)
    rho, u = _fields(dims, seed=grid)
    a = run_gpu("D3Q19", dims, 0.57, "fp32", rho, u, 14, kernel="columns", grid=grid)
    b = run_gpu("D3Q19", dims, 0.57, "fp32", rho, u, 14, kernel="scalar")
    assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])


def test_columns_refusals_and_the_default_choice():
    from paper_2002_02503_amd import lbm

    for lattice, dims in [("D2Q9", (64, 64, 1)), ("D3Q39", (64, 32, 4))]:
        with pytest.raises(lbm.LBMError) as e:
            lbm.Simulation(lattice, dims, 0.6, kernel="columns", torch_memory=False)
        assert e.value.name == "LBM_EINVAL"
    names = {v: k for k, v in lbm.KERNELS.items()}
    for dims, dtype, want in [((201, 150, 77), "fp32", "columns"), ((100, 100, 100), "fp64", "columns"),
                              ((201, 150, 77), "bf16", "columns"), ((128, 128, 128), "fp16", "scalar"),
                              ((101, 101, 101), "fp16", "scalar"), ((700, 700, 1), "fp32", "scalar"),
                              ((100000, 2, 2), "fp32", "scalar"), ((65, 65, 65), "fp32", "scalar")]:
        with lbm.Simulation("D3Q19", dims, 0.8, dtype=dtype, torch_memory=False) as sim:
            assert names[sim.info()["kernel"]] == want, (dims, dtype)


def _batch(lattice, dims, taus, dtype, seed, steps, kernel, **kw):
    from paper_2002_02503_amd import lbm

    rng = np.random.default_rng(seed)
    n = sum(a * b * c for a, b, c in dims)
    rho, u = 1.0 + rng.uniform(-0.01, 0.01, size=n), rng.uniform(-0.05, 0.05, size=(3, n))
    with lbm.Simulation(lattice, dims, taus, dtype=dtype, kernel=kernel, **kw) as sim:
        sim.init(rho, u)
        out = []
        for k in steps:
            out += sim.step(k).moments()
        return out + [sim.get_state()]


BATCHES = [
    # whole rows and pieces of them, sides of one to three sites, several columns a box
    ("D3Q19", [(40, 37, 9), (1, 1, 1), (2, 3, 5), (3, 2, 1), (200, 11, 4), (64, 30, 6)], "fp32", {"theta": 0.5}),
    ("D3Q19", [(40, 37, 9), (7, 5, 300), (129, 6, 3)], "fp64", {}),
    ("D3Q19", [(16, 64, 20), (33, 17, 9)], "fp16", {"K": 2}),
    ("D3Q15", [(20, 30, 10), (61, 29, 8)], "bf16", {"collision": "bgk"}),
    # more planes than blocks: two runs a block
    ("D3Q15", [(5, 4, 40 + k % 3) for k in range(300)], "fp32", {}),
]


@pytest.mark.parametrize("lattice,dims,dtype,kw", BATCHES)
def test_batched_columns_equal_the_one_step_kernel(lattice, dims, dtype, kw):
    """The same bits and checkpoints after odd and even counts, in graphs
    replayed around reads of the state."""
    taus = [0.55 + 0.01 * (k % 40) for k in range(len(dims))]
    a = _batch(lattice, dims, taus, dtype, len(dims), (1, 2, 9, 8), "columns", graph_chunk=4, **kw)
    b = _batch(lattice, dims, taus, dtype, len(dims), (1, 2, 9, 8), "scalar", graph_chunk=1, **kw)
    assert all(np.array_equal(x, y) for x, y in zip(a, b))


def test_batched_columns_choice():
    from paper_2002_02503_amd import lbm

    def kernel_of(lattice, dims, dtype, **kw):
        with lbm.Simulation(lattice, dims, [0.7] * len(dims), dtype=dtype, torch_memory=False, **kw) as sim:
            return {v: k for k, v in lbm.KERNELS.items()}[sim.info()["kernel"]]

    big, small = [(60, 50, 40)] * 8, [(20, 20, 20)] * 200
    assert kernel_of("D3Q19", big, "fp32") == "columns" and kernel_of("D3Q19", big, "fp64") == "columns"
    assert kernel_of("D3Q19", big, "fp16") == "scalar" and kernel_of("D3Q19", small, "fp32") == "scalar"
    assert kernel_of("D3Q19", big, "fp32", block=128) == "scalar" and kernel_of("D3Q39", big, "fp32") == "scalar"
    with pytest.raises(lbm.LBMError) as e:
        lbm.Simulation("D3Q39", [(8, 8, 8), (9, 9, 9)], [0.6, 0.7], kernel="columns", torch_memory=False)
    assert e.value.name == "LBM_EINVAL"


@pytest.mark.parametrize("dims", [(110, 7, 5), (111, 7, 5), (120, 9, 4), (128, 1, 6), (223, 5, 3), (255, 3, 4)])
def test_fp64_columns_at_the_widest_piece(dims):
    """Rows on both sides of the widest FP64 piece (110 sites) and a single row."""
    rho, u = _fields(dims, seed=sum(dims))
    a = run_gpu("D3Q19", dims, 0.6, "fp64", rho, u, 9, kernel="columns")
    b = run_gpu("D3Q19", dims, 0.6, "fp64", rho, u, 9, kernel="scalar")
    assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])


def test_fp64_batched_columns_at_the_widest_piece():
    dims = [(126, 6, 4), (127, 6, 4), (128, 1, 3), (128, 9, 5), (253, 4, 3)]
    a = _batch("D3Q19", dims, [0.6] * len(dims), "fp64", 7, (4, 3), "columns")
    b = _batch("D3Q19", dims, [0.6] * len(dims), "fp64", 7, (4, 3), "scalar")
    assert all(np.array_equal(x, y) for x, y in zip(a, b))


def test_batched_columns_choice_by_shape():
    """Batches whose columns are mostly ring, or too narrow to fill a block, keep
    the one-step kernel."""
    from paper_2002_02503_amd import lbm

    names = {v: k for k, v in lbm.KERNELS.items()}
    for dims, want in [([(1000, 1000, 1)] * 8, "scalar"), ([(4, 4, 5000)] * 60, "scalar"),
                       ([(20000, 2, 2)] * 40, "scalar"), ([(48, 48, 48)] * 64, "columns"),
                       ([(300, 300, 16)] * 8, "columns")]:
        for dtype in ("fp32", "fp64"):
            with lbm.Simulation("D3Q19", dims, [0.7] * len(dims), dtype=dtype, torch_memory=False) as sim:
                assert names[sim.info()["kernel"]] == want, (dims[0], dtype)


def test_16_bit_rows_of_whole_lines_keep_the_one_site_step():
    from paper_2002_02503_amd import lbm

    names = {v: k for k, v in lbm.KERNELS.items()}
    for dims, want in [((256, 250, 64), "scalar"), ((128, 130, 130), "scalar"), ((64, 250, 250), "scalar"),
                       ((130, 130, 130), "columns")]:
        for dtype in ("fp16", "bf16"):
            with lbm.Simulation("D3Q19", dims, 0.8, dtype=dtype, torch_memory=False) as sim:
                assert names[sim.info()["kernel"]] == want, (dims, dtype)
