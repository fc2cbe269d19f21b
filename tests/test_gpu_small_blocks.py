"""Crossbars of at most 64 columns: the one-workgroup Newton-Schulz chains and the
two-chain sweep, at the edges of their 16-column tiles, chain lengths and slabs.

Against the CPU oracle with the float64 tolerance (1e-10: the gate of every float64
solve) and the refinement's (1e-9); the currents-only sweep gives the same bits, and so
does a vector solved alone.
"""
import numpy as np
import pytest

import oracle
import workloads
from tests.gpu_util import TOL_FP64, TOL_IR, gpu_solve, log, node_rel_err, rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 15, 16, 17, 32, 33, 48, 49, 64])
@pytest.mark.parametrize("m,B", [(1, 16), (2, 1), (3, 17), (4, 33), (11, 16), (12, 31)])
def test_small_blocks_match_oracle(m, n, B):
    wl = workloads.random_crossbar(m, n, B, 9000 + 64 * m + n, r_wl=1.5, r_bl=3.0, r_src=40.0, r_sense=60.0)
    log(f"case {wl.name}")
    ref = oracle.solve_workload(wl)
    I, nv, (st, info) = gpu_solve(wl.G, wl.V, wl.geom, ordering="rows")
    assert st == 0 and 0 < info.factor_slots_used <= info.factor_slots_launched
    assert rel_err(I, ref.currents).max() <= TOL_FP64
    assert node_rel_err(nv, ref.node_v).max() <= TOL_FP64
    I2, _, _ = gpu_solve(wl.G, wl.V, wl.geom, node_voltages=False, ordering="rows")
    assert np.array_equal(I, I2)
    k = B - 1
    Ik, nvk, _ = gpu_solve(wl.G, wl.V[k:k + 1], wl.geom, ordering="rows")
    assert np.array_equal(Ik[0], I[k]) and np.array_equal(nvk[0], nv[k])
    If, nvf, (st, _) = gpu_solve(wl.G, wl.V, wl.geom, "fp32_ir", ordering="rows")
    assert st == 0
    assert rel_err(If, ref.currents).max() <= TOL_IR and node_rel_err(nvf, ref.node_v).max() <= TOL_IR


@pytest.mark.parametrize("m,n", [(3, 17), (20, 64)])
def test_small_blocks_of_a_wide_crossbar(m, n):
    """The same sweeps with the inputs on the terminations (reciprocal ordering)."""
    wl = workloads.random_crossbar(m, n, 18, 9900 + n, r_wl=1.5, r_bl=3.0, r_src=40.0, r_sense=60.0)
    ref = oracle.solve_workload(wl)
    I, nv, (st, _) = gpu_solve(wl.G, wl.V, wl.geom, ordering="smaller")
    assert st == 0
    assert rel_err(I, ref.currents).max() <= TOL_FP64 and node_rel_err(nv, ref.node_v).max() <= TOL_FP64


@pytest.mark.parametrize("precision", ["fp64", "fp32_ir"])
@pytest.mark.parametrize("m,n", [(1, 65), (2, 128), (3, 113), (4, 81), (9, 127), (12, 96), (1, 129), (2, 192), (5, 256),
                                 (4, 320)])
def test_shared_launch_factor_matches_oracle(m, n, precision):
    """Factors whose two chains share their launches (column panels at 65 to 128 columns,
    the slot schedule to 320): chains of no, one and a few rows, and devices strong enough
    to need more than one round in a row."""
    for strong in (False, True):
        wl = workloads.random_crossbar(m, n, 5, 9700 + 64 * m + n, r_wl=1.5, r_bl=3.0, r_src=40.0, r_sense=60.0)
        if strong:
            wl.G[:] *= 20.0
        log(f"case {wl.name} {precision} strong={strong}")
        ref = oracle.solve_workload(wl)
        tol = TOL_FP64 if precision == "fp64" else TOL_IR
        outs = []
        for method in ("auto", "checked", "gj"):
            I, nv, (st, info) = gpu_solve(wl.G, wl.V, wl.geom, precision, ordering="rows", factor_method=method)
            assert st == 0 and 0.0 < info.min_pivot
            assert rel_err(I, ref.currents).max() <= tol and node_rel_err(nv, ref.node_v).max() <= tol
            outs.append(I)
        assert np.array_equal(outs[0], outs[1])


@pytest.mark.parametrize("method", ["ns", "checked"])
@pytest.mark.parametrize("n", [16, 64, 65])
def test_checked_factors_wait_for_their_outcome(n, method):
    """Both methods synchronise the plan's stream at every block size, also behind work
    that is still queued there."""
    import torch

    import paper_2410_19993_amd as xb
    wl = workloads.random_crossbar(9, n, 1, 9950 + n)
    G = torch.from_numpy(wl.G).cuda()
    s = torch.cuda.Stream()
    a = torch.randn((4096, 4096), dtype=torch.float64, device="cuda")
    torch.cuda.synchronize()
    log(f"case {method} n={n}")
    with xb.Plan(9, n, 2.5, 2.5, 50.0, 50.0, "fp64", max_batch=1, stream=s, ordering="rows",
                 factor_method=method) as p:
        for _ in range(2):
            with torch.cuda.stream(s):
                p.assemble(G)
                for _ in range(20):
                    a @ a                                  # tens of milliseconds
                p.factor()
                assert s.query()
        assert p.info()[0] == 0
