"""Batched small crossbars: the Newton-Schulz rounds and the elimination of a row.

A row's inverse is found from the row before's by one to three rounds, or by elimination
where the rows differ too much (and in the first row).  Devices of 1 to 100 uS take one
round, twenty times stronger ones two, alternating rows two and an elimination at the
last row; every third row of strong devices is eliminated and the row after it starts
from that inverse.  Shapes: both sides of each padded block size, of a segment of eight
columns, of the 32 rows whose chains are walked together, and of the groups of 16
vectors a wave owns.

Against the oracle with the float64 tolerance of every solve (1e-10).
"""
import numpy as np
import pytest

import oracle
from tests.gpu_util import TOL_FP64, log, rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["weak", "strong", "alternating", "third"])
@pytest.mark.parametrize("m,n,B", [(1, 64, 16), (2, 9, 1), (9, 8, 129), (12, 1, 17), (31, 16, 64), (32, 17, 65),
                                   (33, 31, 256), (12, 32, 128), (34, 33, 15), (65, 64, 256), (7, 57, 100)])
def test_rounds_and_elimination_match_oracle(m, n, B, kind):
    import torch

    import paper_2410_19993_amd as xb
    log(f"case tiles {m}x{n} B={B} {kind}")
    rng = np.random.default_rng(100 * m + n)
    G = np.exp(rng.uniform(np.log(1e-6), np.log(1e-4), (2, m, n)))
    if kind == "strong":
        G *= 20.0
    elif kind == "alternating":
        G[:, 1::2] *= 300.0
    elif kind == "third":
        G[:, 2::3] *= 2e4
    V = rng.uniform(0.0, 0.5, (2, B, m))
    r = (1.5, 3.0, 40.0, 60.0)
    I = xb.tiles_currents(torch.from_numpy(G).cuda(), torch.from_numpy(V).cuda(), *r).cpu().numpy()
    for t in range(2):
        assert rel_err(I[t], oracle.solve(G[t], V[t], *r).currents).max() <= TOL_FP64


@pytest.mark.parametrize("count,m,n", [(57, 4, 130), (58, 4, 130), (33, 5, 200)])
def test_column_and_tile_workgroups_give_the_same_bits(count, m, n):
    """The batched block factor on both sides of its rule (1024 tile workgroups a launch):
    every crossbar of the batch as if it were alone."""
    import torch

    from paper_2410_19993_amd.tiles import TileBatch, TileConfig
    rng = np.random.default_rng(count + n)
    G = torch.from_numpy(np.exp(rng.uniform(np.log(1e-6), np.log(1e-4), (count, m, n)))).cuda()
    V = torch.from_numpy(rng.uniform(0.0, 0.5, (count, 5, m))).cuda()
    r = (1.5, 3.0, 40.0, 60.0)

    def run(G, V):
        batch = TileBatch([(m, n, G.shape[0], 5)], *r, configs=[TileConfig("pipeline")], streams=1)
        out = batch.run([G], [V])[0].cpu().numpy()
        batch.close()
        return out
    out = run(G, V)
    for t in (0, 7, 8, count - 1):
        assert np.array_equal(run(G[t:t + 1].contiguous(), V[t:t + 1].contiguous())[0], out[t])
    assert rel_err(out[1], oracle.solve(G[1].cpu().numpy(), V[1].cpu().numpy(), *r).currents).max() <= TOL_FP64


@pytest.mark.parametrize("n", [1, 8, 16, 17, 32, 33, 64])
def test_rounds_keep_the_pivot_check(n):
    """A row block whose pivots are not positive gives NaN currents also in rows after the
    first.  Devices of 2^60 S swallow the wire conductances: with r_wl = 10 kohm,
    S_1 = -g_bl^2 H_0 - (couplings of 1e-4 S) exactly, a negative diagonal of -1/3 S, whose
    inverse Newton-Schulz rounds find as readily as that of a positive block.  A negative
    pivot would make a current of positive inputs negative.  The other crossbars of the
    call are unaffected."""
    import torch

    import paper_2410_19993_amd as xb
    log(f"case pivot sign n={n}")
    rng = np.random.default_rng(n)
    m, B, r = 4, 3, (1e4, 3.0, 40.0, 60.0)
    G = np.exp(rng.uniform(np.log(1e-6), np.log(1e-4), (5, m, n)))
    G[1, 1], G[2, 2], G[3, 3] = 2.0 ** 60, 2.0 ** 60, 2.0 ** 60
    V = rng.uniform(0.1, 0.5, (5, B, m))
    I = xb.tiles_currents(torch.from_numpy(G).cuda(), torch.from_numpy(V).cuda(), *r).cpu().numpy()
    for t in (0, 4):
        assert rel_err(I[t], oracle.solve(G[t], V[t], *r).currents).max() <= TOL_FP64
    for t in (1, 2, 3):
        assert np.isnan(I[t]).all(), t
