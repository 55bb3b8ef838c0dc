"""Steps captured by the caller into a graph of its own: replays continue the run
with any step kernel, also where one launch takes several steps and an even
number of steps is an odd number of launches, with eager steps and reads between
the replays."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [2, 4, 6, 14, 30])
@pytest.mark.parametrize("kernel,dims", [("scalar", (16, 8, 4)), ("tile", (16, 8, 4)), ("two_step", (64, 8, 4)),
                                         ("columns", (21, 10, 6)), ("columns", [(20, 9, 5), (16, 16, 4)]),
                                         ("auto", (24, 24, 24))])
def test_captured_steps_replay(kernel, dims, n):
    import torch
    from paper_2002_02503_amd import lbm

    rng = np.random.default_rng(n)
    boxes = dims if isinstance(dims, list) else [dims]
    nx, ny, nz = boxes[0]
    tau = [0.6] * len(boxes) if isinstance(dims, list) else 0.6
    sites = sum(int(np.prod(b)) for b in boxes)
    shape = (sites,) if isinstance(dims, list) else (nz, ny, nx)
    rho = 1.0 + rng.uniform(-0.01, 0.01, size=shape)
    u = rng.uniform(-0.05, 0.05, size=(3,) + shape)
    s = torch.cuda.Stream()
    with torch.cuda.stream(s), \
            lbm.Simulation("D3Q19", dims, tau, dtype="fp32", kernel=kernel, stream=s) as a, \
            lbm.Simulation("D3Q19", dims, tau, dtype="fp32", kernel="scalar", graph_chunk=1, stream=s) as b:
        a.init(rho, u).step(3)
        b.init(rho, u).step(3)
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            a.step(n)
        for eager in (2, 8, 36):
            g.replay()
            b.step(n)
            ra, rb = a.moments(), b.moments()
            assert np.array_equal(ra[0], rb[0]) and np.array_equal(ra[1], rb[1])
            a.step(eager)
            b.step(eager)
            ra, rb = a.moments(), b.moments()
            assert np.array_equal(ra[0], rb[0]) and np.array_equal(ra[1], rb[1])


BOXES = [("scalar", (16, 8, 4)), ("tile", (16, 8, 4)), ("two_step", (64, 8, 4)), ("columns", (21, 10, 6)),
         ("columns", [(20, 9, 5), (16, 16, 4)]), ("auto", (24, 24, 24)), ("auto", (64, 64, 64))]


def _state(dims, seed):
    rng = np.random.default_rng(seed)
    boxes = dims if isinstance(dims, list) else [dims]
    nx, ny, nz = boxes[0]
    tau = [0.6] * len(boxes) if isinstance(dims, list) else 0.6
    shape = (sum(int(np.prod(b)) for b in boxes),) if isinstance(dims, list) else (nz, ny, nx)
    return tau, 1.0 + rng.uniform(-0.01, 0.01, size=shape), rng.uniform(-0.05, 0.05, size=(3,) + shape)


def _same(a, b):
    ra, rb = a.moments(), b.moments()
    return np.array_equal(ra[0], rb[0]) and np.array_equal(ra[1], rb[1])


@pytest.mark.parametrize("warm", [2, 8])
@pytest.mark.parametrize("kernel,dims", BOXES)
def test_new_fields_after_a_capture(kernel, dims, warm):
    """Steps captured after warm-up steps, then replayed on other fields
    (lbm_init) and on a checkpoint (lbm_set_state)."""
    import torch
    from paper_2002_02503_amd import lbm

    tau, rho, u = _state(dims, 1)
    _, rho2, u2 = _state(dims, 2)
    s = torch.cuda.Stream()
    with torch.cuda.stream(s), \
            lbm.Simulation("D3Q19", dims, tau, dtype="fp32", kernel=kernel, stream=s) as a, \
            lbm.Simulation("D3Q19", dims, tau, dtype="fp32", kernel="scalar", graph_chunk=1, stream=s) as b:
        a.init(rho, u).step(warm)
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            a.step(2)
        for r, v in ((rho2, u2), (rho, u)):
            a.init(r, v)
            b.init(r, v)
            for eager in (0, 2, 34):
                a.step(eager)
                b.step(eager)
                g.replay()
                b.step(2)
                assert _same(a, b)
        ck = b.get_state()
        a.step(6)
        a.set_state(ck)
        g.replay()
        b.step(2)
        assert _same(a, b)


@pytest.mark.parametrize("warm", [2, 8])
@pytest.mark.parametrize("kernel,dims", BOXES)
def test_captured_reader(kernel, dims, warm):
    """A captured lbm_residual_noalloc reports the current state after even
    numbers of eager steps and after new fields."""
    import torch
    from paper_2002_02503_amd import lbm

    tau, rho, u = _state(dims, 3)
    _, rho2, u2 = _state(dims, 4)
    s = torch.cuda.Stream()
    with torch.cuda.stream(s), \
            lbm.Simulation("D3Q19", dims, tau, dtype="fp32", kernel=kernel, stream=s) as a:
        dr, du = torch.from_numpy(rho).cuda(), torch.from_numpy(u).cuda()
        out, ref = torch.zeros(4, dtype=torch.float64, device="cuda"), torch.zeros(4, dtype=torch.float64, device="cuda")
        a.init(rho, u).step(warm)
        s.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            a.residual_noalloc(dr, du, out)
        for eager in (2, 2, 8, 34):
            a.step(eager)
            g.replay()
            a.residual_noalloc(dr, du, ref)
            assert torch.equal(out, ref) and float(ref[0]) > 0.0
        a.init(rho2, u2).step(4)
        g.replay()
        a.residual_noalloc(dr, du, ref)
        assert torch.equal(out, ref)


@pytest.mark.parametrize("chunk,n", [(None, 32), (None, 64), (None, 70), (4, 8), (4, 10), (2, 6)])
@pytest.mark.parametrize("prepared", [False, True])
@pytest.mark.parametrize("kernel,dims", BOXES)
def test_captured_steps_of_a_graph_chunk_and_more(kernel, dims, prepared, chunk, n):
    """Captured counts at and above the handle's own graph chunk, whose graphs
    exist (prepared) or not."""
    import torch
    from paper_2002_02503_amd import lbm

    tau, rho, u = _state(dims, 5)
    s = torch.cuda.Stream()
    with torch.cuda.stream(s), \
            lbm.Simulation("D3Q19", dims, tau, dtype="fp32", kernel=kernel, stream=s, graph_chunk=chunk) as a, \
            lbm.Simulation("D3Q19", dims, tau, dtype="fp32", kernel="scalar", graph_chunk=1, stream=s) as b:
        a.init(rho, u).step(2)
        b.init(rho, u).step(2)
        if prepared:
            a.prepare()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            a.step(n)
        for eager in (0, 2, 40):
            g.replay()
            b.step(n)
            assert _same(a, b)
            a.step(eager)
            b.step(eager)
            assert _same(a, b)
