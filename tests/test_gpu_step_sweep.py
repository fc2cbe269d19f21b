"""Substitution as one launch per step of the two chains (more than 64 columns, batches
that leave most of the GPU idle in the slab sweep), at every block size and choice of
waves and slabs per workgroup, chain lengths of one to a few rows, and partial slabs.

Against the CPU oracle within the float64 tolerance (1e-10: the gate of every float64
solve), and bit for bit against the slab sweep, which a batch too large for the step path
takes: an input vector's results do not depend on what shares its batch.
"""
import numpy as np
import pytest

import oracle
import workloads
from tests.gpu_util import TOL_FP64, TOL_IR, gpu_solve, log, node_rel_err, rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n,B,seed", [
    (3, 65, 1, 1), (4, 128, 17, 2), (7, 129, 200, 3), (8, 192, 40, 4), (9, 250, 90, 5), (6, 320, 150, 6),
    (5, 383, 33, 7), (12, 448, 20, 8), (10, 512, 16, 9), (3, 512, 129, 10)])
def test_step_sweep_matches_oracle(m, n, B, seed):
    wl = workloads.random_crossbar(m, n, B, 7700 + seed, r_wl=1.5, r_bl=3.0, r_src=40.0, r_sense=60.0)
    log(f"case {wl.name}")
    ref = oracle.solve_workload(wl)
    I, nv, (st, _) = gpu_solve(wl.G, wl.V, wl.geom, ordering="rows")
    assert st == 0
    assert rel_err(I, ref.currents).max() <= TOL_FP64 and node_rel_err(nv, ref.node_v).max() <= TOL_FP64
    I2, _, _ = gpu_solve(wl.G, wl.V, wl.geom, node_voltages=False, ordering="rows")
    assert np.array_equal(I, I2)


@pytest.mark.parametrize("m,n", [(5, 512), (6, 300), (7, 128)])
def test_step_sweep_same_bits_as_slab_sweep(m, n):
    """The same vectors inside a batch past the step path's limit and in batches that take
    each of its layouts."""
    B = 16 * 129                       # past the step path and the chain per workgroup
    wl = workloads.random_crossbar(m, n, B, 7800 + n)
    log(f"case {wl.name}")
    I, nv, (st, _) = gpu_solve(wl.G, wl.V, wl.geom, ordering="rows")
    assert st == 0
    for k in (1, 17, 16 * 20 + 3, 16 * 64, 16 * 65, B - 16):
        Ik, nvk, _ = gpu_solve(wl.G, wl.V[:k], wl.geom, ordering="rows")
        assert np.array_equal(Ik, I[:k]) and np.array_equal(nvk, nv[:k]), f"batch of {k}"


def test_step_sweep_of_a_wide_crossbar():
    """Inputs on the terminations (reciprocal ordering)."""
    wl = workloads.random_crossbar(70, 90, 21, 7900, r_wl=1.5, r_bl=3.0, r_src=40.0, r_sense=60.0)
    ref = oracle.solve_workload(wl)
    I, nv, (st, _) = gpu_solve(wl.G, wl.V, wl.geom, ordering="smaller")
    assert st == 0
    assert rel_err(I, ref.currents).max() <= TOL_FP64 and node_rel_err(nv, ref.node_v).max() <= TOL_FP64


@pytest.mark.parametrize("m,n,B,seed", [(3, 129, 1, 1), (6, 250, 130, 2), (7, 320, 48, 3), (9, 512, 300, 4)])
def test_refinement_by_steps(m, n, B, seed):
    """The refinement's float32 sweeps by steps: within the refinement's tolerance (1e-9),
    and the bits and sweep count of the slab sweep, which a larger batch takes."""
    wl = workloads.random_crossbar(m, n, B, 7950 + seed, r_wl=1.5, r_bl=3.0, r_src=40.0, r_sense=60.0)
    log(f"case {wl.name} fp32_ir")
    ref = oracle.solve_workload(wl)
    I, nv, (st, info) = gpu_solve(wl.G, wl.V, wl.geom, "fp32_ir", ordering="rows")
    assert st == 0
    assert rel_err(I, ref.currents).max() <= TOL_IR and node_rel_err(nv, ref.node_v).max() <= TOL_IR
    V = np.tile(wl.V, (-(-(16 * 128 + 1) // B), 1))
    Ib, nvb, (stb, infob) = gpu_solve(wl.G, V, wl.geom, "fp32_ir", ordering="rows")
    assert stb == 0 and infob.ir_iters == info.ir_iters
    k = B // 16 * 16                   # a slab stops as a whole: compare whole ones
    assert np.array_equal(Ib[:k], I[:k]) and np.array_equal(nvb[:k], nv[:k])


@pytest.mark.parametrize("m,n", [(1, 64), (16, 129), (256, 70), (257, 64), (257, 130)])
def test_transfer_by_either_route(m, n):
    """T by unit solves (one batch holds them, few rows or columns) and by the block
    recurrences (the last shape, and a plan whose batch is one row short): both against
    the oracle, and the last solve's backward error is reported after either."""
    import torch

    import paper_2410_19993_amd as xb
    wl = workloads.random_crossbar(m, n, 3, 8800 + m + n, r_wl=1.5, r_bl=3.0, r_src=40.0, r_sense=60.0)
    g = wl.geom
    ref = oracle.solve(wl.G, np.eye(m), g.r_wl, g.r_bl, g.r_src, g.r_sense).currents
    for max_batch in (max(m, 256), max(m - 1, 64)):
        log(f"case transfer {m}x{n} max_batch={max_batch}")
        with xb.Plan(m, n, g.r_wl, g.r_bl, g.r_src, g.r_sense, "fp64", max_batch=max_batch, ordering="rows") as p:
            p.assemble(torch.from_numpy(wl.G).cuda())
            p.factor()
            before = p.info()[1].max_backward_err
            T = p.transfer().cpu().numpy()
            st, info = p.info()
        assert st == 0 and info.max_backward_err == before
        assert rel_err(T, ref).max() <= TOL_FP64


@pytest.mark.parametrize("precision", ["fp64", "fp32_ir"])
@pytest.mark.parametrize("m,n", [(20, 50), (12, 30), (9, 200)])
def test_captured_pass_replays_the_eager_bits(m, n, precision):
    """Assembly, factor, solve, currents and transfer of the small-block and step paths in
    one graph: every replay, with eager work between, gives the eager bits."""
    import torch

    import paper_2410_19993_amd as xb
    wl = workloads.random_crossbar(m, n, 18, 8600 + n, r_wl=2.5, r_bl=2.5)
    G, V = torch.from_numpy(wl.G).cuda(), torch.from_numpy(np.ascontiguousarray(wl.V)).cuda()
    nv = torch.empty((18, 2 * m * n), dtype=torch.float64, device="cuda")
    I = torch.empty((18, n), dtype=torch.float64, device="cuda")
    T = torch.empty((m, n), dtype=torch.float64, device="cuda")
    s = torch.cuda.Stream()
    log(f"case capture {m}x{n} {precision}")
    with xb.Plan(m, n, 2.5, 2.5, 50.0, 50.0, precision, max_batch=32, stream=s, ordering="rows") as p:
        def step():
            p.assemble(G)
            p.factor()
            p.solve_batch(V, nv)
            p.currents(I)
            p.transfer(T)
        with torch.cuda.stream(s):
            step()
        s.synchronize()
        eager = [x.clone() for x in (I, nv, T)]
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=s):
            step()
        for _ in range(3):
            for x in (I, nv, T):
                x.fill_(-1.0)
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            assert all(torch.equal(x, e) for x, e in zip((I, nv, T), eager))
            with torch.cuda.stream(s):
                p.assemble(G * 1.01)
                p.factor()
            s.synchronize()
        st, _ = p.info()
    assert st == 0
    assert rel_err(eager[0].cpu().numpy(), oracle.solve_workload(wl).currents).max() <= (
        TOL_FP64 if precision == "fp64" else TOL_IR)


def _graph_nodes(graph):
    """Number of nodes of a captured torch graph."""
    import ctypes
    with open("/proc/self/maps") as f:
        path = next(line.split()[-1] for line in f if "libamdhip64" in line)
    nodes = ctypes.c_size_t(0)
    assert ctypes.CDLL(path).hipGraphGetNodes(ctypes.c_void_p(graph.raw_cuda_graph()), None, ctypes.byref(nodes)) == 0
    return nodes.value


@pytest.mark.parametrize("m,n,B,tol,sweeps", [(3, 192, 16, 1e-3, 3), (8, 192, 16, 1e-6, 4), (3, 192, 2048, 0.0, 3),
                                              (64, 256, 2048, 1e-6, 2), (3, 512, 16, 0.0, 6)])
def test_refinement_queues_few_idle_steps(m, n, B, tol, sweeps):
    """Launches that a refinement queues: m + 3 for each of its first `sweeps` sweeps (two
    panels formed, m / 2 forward, the twist, m / 2 back, the decision; m rounded up to even),
    one for each later sweep, one for each residual, one to clear the slabs' state.  A short
    chain or a loose tolerance does not queue long runs of steps that find nothing to do."""
    import torch

    import paper_2410_19993_amd as xb
    wl = workloads.random_crossbar(m, n, B, 8650 + n, r_wl=2.5, r_bl=2.5)
    G, V = torch.from_numpy(wl.G).cuda(), torch.from_numpy(wl.V).cuda()
    s = torch.cuda.Stream()
    log(f"case {wl.name} tol={tol}")
    with xb.Plan(m, n, 2.5, 2.5, 50.0, 50.0, "fp32_ir", max_batch=B, ir_tol=tol, ir_max_iter=10, stream=s,
                 ordering="rows") as p:
        with torch.cuda.stream(s):
            p.assemble(G)
            p.factor()
            p.solve_batch(V)
        s.synchronize()
        graph = torch.cuda.CUDAGraph(keep_graph=True)
        with torch.cuda.graph(graph, stream=s):
            p.solve_batch(V)
        st, info = p.info()
        I = p.currents().cpu().numpy()
    log(f"   {info.ir_iters} sweeps, {_graph_nodes(graph)} launches")
    g = wl.geom
    ref = oracle.solve(wl.G, wl.V[:2], g.r_wl, g.r_bl, g.r_src, g.r_sense).currents
    assert st == 0 and rel_err(I[:2], ref).max() <= max(TOL_IR, 10 * tol)
    per_sweep = 2 + 2 * (m // 2) + 1 + 1
    assert _graph_nodes(graph) <= sweeps * per_sweep + (11 - sweeps) + 10 + 1


@pytest.mark.parametrize("m,n,B", [(24, 192, 33), (16, 320, 16), (9, 448, 20)])
def test_refinement_past_the_steps(m, n, B):
    """A solve that is not finished when its sweeps by steps end: the slab sweep goes on from
    their state (solution buffer, residual, last corrections) to the same bits and count as
    when it runs alone, in a batch past the steps' limit, and to the oracle's currents.  A
    bfloat16 factor gains about two digits a sweep."""
    wl = workloads.random_crossbar(m, n, B, 8000 + n, r_wl=1.5, r_bl=3.0, r_src=40.0, r_sense=60.0)
    log(f"case {wl.name} bf16_ir")
    kw = dict(precision="bf16_ir", ordering="rows", ir_max_iter=40)
    I, nv, (st, info) = gpu_solve(wl.G, wl.V, wl.geom, **kw)
    log(f"   status {st}, {info.ir_iters} sweeps")
    assert st == 0 and info.ir_iters > 6
    ref = oracle.solve_workload(wl)
    assert rel_err(I, ref.currents).max() <= TOL_IR and node_rel_err(nv, ref.node_v).max() <= TOL_IR
    V = np.tile(wl.V, (-(-(16 * 128 + 1) // B), 1))
    Ib, nvb, (stb, infob) = gpu_solve(wl.G, V, wl.geom, **kw)
    assert stb == 0 and infob.ir_iters >= info.ir_iters    # (its slabs hold other vectors too)
    k = B // 16 * 16
    assert np.array_equal(Ib[:k], I[:k]) and np.array_equal(nvb[:k], nv[:k])


@pytest.mark.parametrize("n", [192, 512])
def test_refinement_by_steps_reports_non_convergence(n):
    """One correction sweep cannot reach a 1e-15 estimate: the steps' decision flags it as the
    slab sweep's does, and leaves the last solution."""
    from paper_2410_19993_amd import _lib
    B = 20
    wl = workloads.random_crossbar(12, n, B, 8050 + n)
    log(f"case {wl.name} fp32_ir, one correction")
    kw = dict(precision="fp32_ir", ordering="rows", ir_tol=1e-15, ir_max_iter=1)
    I, nv, (st, info) = gpu_solve(wl.G, wl.V, wl.geom, **kw)
    assert st == _lib.XBAR_ERR_NO_CONVERGENCE and info.ir_iters == 2
    Ib, nvb, (st, info) = gpu_solve(wl.G, np.tile(wl.V, (103, 1)), wl.geom, **kw)
    assert st == _lib.XBAR_ERR_NO_CONVERGENCE and info.ir_iters == 2
    assert np.array_equal(Ib[:B], I) and np.array_equal(nvb[:B], nv)


@pytest.mark.parametrize("m,n", [(16, 129), (40, 40), (257, 130)])
def test_transfer_keeps_the_last_backward_error(m, n):
    """The backward error of the last solve is still reported after a transfer by unit
    solves (the first two shapes) and by the block recurrences (the last)."""
    import torch

    import paper_2410_19993_amd as xb
    wl = workloads.random_crossbar(m, n, 3, 8850 + m + n)
    log(f"case backward error, transfer {m}x{n}")
    with xb.Plan(m, n, 2.5, 2.5, 50.0, 50.0, "fp64", max_batch=max(m, 256), ordering="rows") as p:
        p.set_diagnostics(True)
        p.assemble(torch.from_numpy(wl.G).cuda())
        p.factor()
        p.solve_batch(torch.from_numpy(wl.V).cuda(), torch.empty((3, 2 * m * n), dtype=torch.float64, device="cuda"))
        before = p.info()[1].max_backward_err
        p.transfer()
        st, info = p.info()
    assert st == 0 and 0.0 <= before <= 1e-12 and info.max_backward_err == before
