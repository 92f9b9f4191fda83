"""Exterior moments and the folded near-field operators (host tables): for
random leaf values the potentials formed from folded values and moments equal
the products with the near-field tables, for every configuration.  Tolerance:
the tables' own quadrature error (2e-14 of the largest entry, pinned against
the oracle in test_library_host.py) summed over the K^2 products."""
import numpy as np
import pytest

from paper_2211_14537_amd import vfx


def fold(f, K, q):
    sx, sy = (-1.0 if q & 2 else 1.0), (-1.0 if q & 1 else 1.0)
    F = f.reshape(K, K)
    G = F + sy * F[:, ::-1] + sx * F[::-1] + sx * sy * F[::-1, ::-1]
    return G[:K // 2, :K // 2].ravel()


def unfold(y, K):
    H = K // 2
    out = np.zeros((K, K))
    for q in range(4):
        sx, sy = (-1.0 if q & 2 else 1.0), (-1.0 if q & 1 else 1.0)
        Y = y[q].reshape(H, H)
        out[:H, :H] += Y
        out[:H, H:] += sy * Y[:, ::-1]
        out[H:, :H] += sx * Y[::-1]
        out[H:, H:] += sx * sy * Y[::-1, ::-1]
    return out.ravel()


@pytest.mark.parametrize("K,p", [(4, 9), (8, 20), (12, 30), (16, 24), (16, 60)])
def test_moment_operators_match_the_near_tables(K, p):
    ctx = vfx.Context(K, p)
    n, H2, P = K * K, K * K // 4, p + 1
    E, SH = 2 * K - 4, K * K // 16
    SE, R = E // 4, 16 * ((H2 + 15) // 16)
    KS = SH + 8 * SE
    V = ctx.debug_table(29, 0, 4 * H2 * E).reshape(4, H2, E)
    rows = 16 * ((E + (P + 1) // 2 + 15) // 16)
    momT = ctx.debug_table(30, 0, 4 * H2 * rows).reshape(4, SH, 4, rows).transpose(0, 2, 1, 3).reshape(4, H2, rows)
    symT = ctx.debug_table(31, 0, 4 * KS * 4 * R).reshape(4, KS, 4, R)
    pairT = ctx.debug_table(32, 0, 24 * 4 * E * n).reshape(24, 4, SE, 4, n).transpose(0, 1, 3, 2, 4).reshape(24, 4, E, n)
    near = [ctx.debug_table(0, c, n * n).reshape(n, n).T for c in range(33)]
    p2m = ctx.debug_table(2, 0, 2 * P * n).reshape(P, n, 2)
    for q in range(4):  # orthonormal bases
        assert np.abs(V[q].T @ V[q] - np.eye(E)).max() < 1e-14
    rng = np.random.default_rng(K)
    src = [rng.standard_normal(n) for _ in range(9)]
    fh = [[fold(f, K, q) for q in range(4)] for f in src]
    m = [[V[q].T @ fh[s][q] for q in range(4)] for s in range(9)]
    tol = lambda A: 2e-14 * n * np.abs(A).max() * 4  # noqa: E731
    # multipoles from the folded values
    a = np.zeros((P, 2))
    for q in range(4):
        r = momT[q].T @ fh[0][q]
        assert np.abs(r[:E] - m[0][q]).max() < 1e-13 * n
        l = 2 * np.arange((P + 1) // 2) + (q in (1, 2))
        a[l[l < P], q & 1] = r[E:E + (P + 1) // 2][l < P]
    want = np.einsum("kjc,j->kc", p2m, src[0])
    assert np.abs(a - want).max() < 1e-13 * n * np.abs(p2m).max()
    # coarse and fine neighbours
    for c in range(24):
        y = sum(m[0][q] @ pairT[c, q] for q in range(4))
        assert np.abs(y - near[9 + c] @ src[0]).max() < tol(near[9 + c])
    # own leaf and the eight same-level neighbours together
    cfgs = [4, 7, 1, 5, 3, 8, 2, 6, 0]  # own, +x, -x, +y, -y, ++, -+, +-, --
    ys = []
    for q in range(4):
        qx, qy = q >> 1, q & 1
        sg = lambda p, bit: 1.0 if ((q ^ p) & bit) == 0 else -1.0  # noqa: E731
        col = [fh[0][q].reshape(4, SH)]
        for p in (qy, 2 + qy):
            col.append((m[1][p] + sg(p, 2) * m[2][p]).reshape(4, SE))
        for p in (2 * qx, 2 * qx + 1):
            col.append((m[3][p] + sg(p, 1) * m[4][p]).reshape(4, SE))
        for p in range(4):
            col.append((m[5][p] + sg(p, 2) * m[6][p] + sg(p, 1) * (m[7][p] + sg(p, 2) * m[8][p])).reshape(4, SE))
        ys.append(np.einsum("ls,slr->r", np.concatenate(col, axis=1), symT[q])[:H2])
    y = unfold(ys, K)
    want = sum(near[c] @ src[s] for s, c in enumerate(cfgs))
    assert np.abs(y - want).max() < tol(near[4])
