"""QR/LQ and visit kernels at the edges of their tiles: one message update of
a small block with Gaussian messages that fill the bond cap, so that its inner
panels are (chi D^2) x chi, against the FP64 oracle's column absorptions.  The
bond caps straddle a column block (16, 17, 33, 49), a row tile and the change
from the one-workgroup QR (768 x 48) to the one with a workgroup per column
tile."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# Messages compared as unit vectors, as in the other message tests: the
# oracle moves by 1e-14 to 1e-13 when its inputs move by 1e-15.
TOL = 1e-12


def _message(rng, n, P, chi):
    b = [1] + [min(chi, P ** min(i, n - i)) for i in range(1, n)] + [1]
    m = [rng.standard_normal((b[i], P, b[i + 1])) for i in range(n)]
    return [t / np.linalg.norm(t) for t in m], b


@pytest.mark.parametrize("D,chi", [
    (2, 1), (2, 3), (2, 4), (3, 9), (4, 15), (4, 16),   # one column tile
    (5, 17), (5, 25),                                   # two, D^2 odd
    (6, 21), (6, 22), (6, 33), (6, 36),                 # 756, 792, 1188, 1296 rows
    (7, 49),                                            # 2401 x 49: one column in the last tile
])
def test_panel_edges(D, chi):
    _compare(D, 2, 2, chi)


def _compare(D, H, W, chi):
    import torch
    from oracle import blockbp as ob
    from paper_2301_05844_amd import bbp
    rng = np.random.default_rng(1000 * D + chi)
    P = D * D
    A = 0.3 * rng.standard_normal((H * W, 2, D, D, D, D))
    A[:, 0, 0, 0, 0, 0] += 1.0
    sides = [_message(rng, n, P, chi) for n in (W, H, W)]
    dev = []
    for m, b in sides:
        s = np.zeros((len(m), chi, P, chi))
        for i, t in enumerate(m):
            s[i, :t.shape[0], :, :t.shape[2]] = t
        dev.append((torch.from_numpy(s).cuda(), b))
    out, bonds, scale = bbp.update_message(torch.from_numpy(A).cuda(), *dev, H=H, W=W, D=D,
                                           chi=chi)
    grid = [[A[y * W + x] for x in range(W)] for y in range(H)]
    Y, ls, _, _ = ob.absorb(grid, *[m for m, _ in sides], chi, 2, 0, lambda c: c)
    ref = ob.extract_message(Y)
    assert [int(v) for v in bonds] == [1] + [t.shape[2] for t in ref]
    got = out.cpu().numpy().reshape(H, chi, P, chi)
    got = [got[i, :bonds[i], :, :bonds[i + 1]] for i in range(H)]
    g, r = ob.mps_dense(got), ob.mps_dense(ref)
    assert abs(scale - ls) < TOL
    assert min(np.abs(g - r).max(), np.abs(g + r).max()) < TOL


@pytest.mark.parametrize("D,H,chi", [
    (2, 3, 5), (2, 6, 17), (2, 6, 21), (2, 6, 64),         # X, G tiles of 1, 2, 4 columns
    (3, 4, 9), (3, 4, 16), (3, 4, 17), (3, 4, 33), (3, 4, 49),
    (5, 3, 16), (5, 3, 24),                                 # four xb of one yf
    (5, 4, 33), (5, 4, 37), (6, 4, 33),                     # four yf, the xb range split
])
def test_visit_edges(D, H, chi):
    """Visits at the edges of their tiles: bond caps below, at and above 16
    columns, rows that leave a tile of yf or xb partly empty, and the split of
    the xb range over workgroups."""
    _compare(D, H, 2, chi)


@pytest.mark.parametrize("H,W,chi", [
    (1, 1, 1), (1, 3, 4), (2, 2, 8), (5, 3, 8), (4, 2, 9), (6, 2, 16), (6, 3, 17), (6, 2, 20),
])
def test_small_columns(H, W, chi):
    """The column absorptions that run as one launch (D = 2, bond caps to 20):
    the shortest column, panels for one wave (to 8) and for four, and the
    change from one column tile to two."""
    _compare(2, H, W, chi)


@pytest.mark.parametrize("D,chi", [
    (3, 4), (3, 7), (3, 8), (3, 14), (3, 15),   # 36, 63 | 72, 126 | 135 rows of four waves
    (5, 10), (5, 11),                           # 250 rows | 275 of eight
])
def test_single_column_tile_edges(D, chi):
    _compare(D, 3, 2, chi)


# one item at caps 33 to 48: the D = 4 visit's 1 x 4 pairs, back bonds in
# whole and ragged steps of four
@pytest.mark.parametrize("chi", [33, 36, 42, 48])
def test_small_batch_visit_at_three_column_tiles(chi):
    _compare(4, 4, 2, chi)


@pytest.mark.parametrize("D,H,chi", [
    (4, 6, 48),             # 768 x 48, the largest of one workgroup
    (4, 6, 49), (5, 5, 60), (6, 5, 54),   # 784, 1500 and 1944 rows: a workgroup per column tile
    (6, 5, 86),             # 3096 x 86: beyond those, streamed from global memory
])
def test_tall_panels(D, H, chi):
    """Columns long enough for inner panels of the full (chi D^2) x chi."""
    _compare(D, H, 2, chi)


@pytest.mark.parametrize("chi", [33, 48])
def test_visit_of_three_column_tiles_at_the_smallest_bond(chi):
    _compare(2, 6, 2, chi)


@pytest.mark.parametrize("chi_env", [12, 16, 40])
def test_environments_at_the_smallest_bond(chi_env):
    """D = 2 observables: the pair-per-wave visit without a local update, at one
    and three column tiles, against the oracle (tolerance of the observables)."""
    from bbp_inputs import op_sz, peps_finite
    from oracle import blockbp as ob
    from paper_2301_05844_amd import bbp
    kw = dict(Lx=8, Ly=8, bx=4, by=4, D=2, chi=8, chi_env=chi_env)
    A = peps_finite(8, 8, 2, seed=7)
    ref, g = ob.BlockBP(A, **kw), bbp.BlockBP(**kw)
    g.set_tensors(A)
    for _ in range(3):
        ref.sweep()
        g.sweep()
    xs, ys = [0, 3, 4, 5, 7], [1, 3, 2, 6, 7]
    sz = g.expect_sites(xs, ys, op_sz())
    for i in range(len(xs)):
        assert abs(sz[i] - ref.expect_site(xs[i], ys[i], op_sz())) < 1e-10
