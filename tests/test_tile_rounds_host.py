"""The rule by which the one-workgroup tile kernel inverts a row by rounds (no pivot check)
or eliminates it (csrc/tiles.hip, round_limit), on the host: up to the conductance that it
allows, every S_i that the kernel's recurrences form in float64 is strictly diagonally
dominant with a positive diagonal, so that its pivots are positive; far past it, some are not.
"""
import numpy as np
import pytest


def round_limit(g_bl, g_sense):
    if not (g_bl <= 1e299 and g_sense <= 1e299):
        return -1.0
    return min(1e10 * min(g_bl, g_sense) - g_bl, 1e299)


def blocks(G, g_wl, g_bl, g_src, g_sense):
    """S_0 .. S_{m-1} by the kernel's recurrences: the word-line chain in excess form, T^-1 as
    products of ratios, S_i = diag(q_i) - Gam T^-1 Gam - g_bl^2 S_{i-1}^-1."""
    m, n = G.shape
    H, out = None, []
    for i in range(m):
        g = G[i]
        p, e = np.empty(n), 0.0
        for j in range(n):
            e = g[0] + g_src if j == 0 else g[j] + g_wl * e / p[j - 1]
            p[j] = e + (g_wl if j < n - 1 else 0.0)
        r, d = g_wl / p, np.empty(n)
        d[n - 1] = 1.0 / p[n - 1]
        for k in range(n - 2, -1, -1):
            d[k] = (1.0 / p[k]) * (g_wl * r[k] * d[k + 1] + 1.0)
        T = np.empty((n, n))
        for k in range(n):
            x = d[k]
            T[k, k] = x
            for j in range(k - 1, -1, -1):
                x *= r[j]
                T[j, k] = T[k, j] = x
        S = -(g[:, None] * T) * g[None, :]
        above, below = (g_bl if i > 0 else 0.0), (g_bl if i < m - 1 else g_sense)
        S[np.diag_indices(n)] += g + above + below
        if H is not None:
            S -= g_bl * g_bl * H
        H = np.linalg.inv(S)
        H = 0.5 * (H + H.T)
        out.append(S)
    return out


def dominance(S):
    """Smallest excess of a diagonal entry over its column's other magnitudes."""
    d = np.diag(S)
    return (d - (np.abs(S).sum(axis=0) - np.abs(d))).min()


@pytest.mark.parametrize("r", [(1.5, 3.0, 40.0, 60.0), (1e4, 3.0, 40.0, 60.0), (1e-3, 1e-3, 50.0, 50.0),
                               (1e-6, 3.0, 50.0, 50.0), (2.5, 1e5, 50.0, 50.0), (2.5, 2.5, 50.0, 1e8),
                               (2.5, 2.5, 1e-6, 1e-6)])
@pytest.mark.parametrize("m,n", [(2, 1), (6, 9), (5, 33), (4, 64)])
def test_blocks_within_the_limit_are_dominant(m, n, r):
    g_wl, g_bl, g_src, g_sense = (1.0 / x for x in r)
    top = round_limit(g_bl, g_sense)
    rng = np.random.default_rng(m * n)
    for kind in range(4):
        if kind == 0:
            G = np.exp(rng.uniform(np.log(1e-6), np.log(top), (m, n)))
        elif kind == 1:
            G = np.full((m, n), top)
        elif kind == 2:
            G = np.exp(rng.uniform(np.log(1e-6), np.log(1e-4), (m, n)))
            G[1:, rng.integers(n)] = top * rng.uniform(0.5, 1.0)
        else:
            G = np.exp(rng.uniform(np.log(1e-6), np.log(1e-4), (m, n)))
            G[m // 2] = top * rng.uniform(0.5, 1.0, n)
        for S in blocks(G, g_wl, g_bl, g_src, g_sense):
            assert dominance(S) > 0.0


def test_blocks_far_past_the_limit_are_not():
    g_wl, g_bl, g_src, g_sense = 1e-4, 1 / 3.0, 1 / 40.0, 1 / 60.0
    G = np.full((3, 8), 1e-5)
    G[1] = 2.0 ** 60
    assert G[1, 0] > round_limit(g_bl, g_sense)
    assert dominance(blocks(G, g_wl, g_bl, g_src, g_sense)[1]) < 0.0
