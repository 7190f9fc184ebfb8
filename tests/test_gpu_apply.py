"""GPU parity of Q^T B and Q B on blocks of columns: the products of many columns are formed in
blocks of 16 x 16 (32 x 32 in double double) outputs, those of fewer than 16 columns a wave per
output; both against the oracle's reflectors at the edges of the blocks (tiles, rows and columns
that are no multiple of 16, one more and one less than a block)."""
import numpy as np
import pytest

import mdgen

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def unit(P):
    return 2.0 ** -(53 * P - (P - 1))


def md_err(x, ref):
    d = np.zeros(ref.shape[1:])
    for k in range(ref.shape[0] - 1, -1, -1):
        d = d + (x[k] - ref[k])
    return np.max(np.abs(d)) / np.max(np.abs(ref[0]))


CASES = [
    # P, m, n, tile, columns of B
    (2, 300, 96, 48, 33), (2, 65, 40, 20, 16), (2, 70, 64, 64, 15), (2, 45, 45, 45, 32), (2, 40, 31, 31, 1),
    (4, 90, 60, 20, 17), (4, 130, 100, 100, 64), (4, 260, 256, 256, 31), (4, 33, 9, 1, 18),
    (8, 50, 24, 12, 16), (8, 40, 33, 33, 40), (8, 70, 64, 64, 3), (1, 100, 48, 16, 50),
]


@pytest.mark.parametrize("P,m,n,tile,nrhs", CASES)
def test_apply_block_of_columns(orc, P, m, n, tile, nrhs):
    import paper_2110_08375_amd as M

    print("case apply P=%d m=%d n=%d tile=%d nrhs=%d" % (P, m, n, tile, nrhs), flush=True)
    A = mdgen.md_uniform(P, m, n, 500 + m, mdgen.STREAM_A)
    B = mdgen.md_uniform(P, m, nrhs, 600 + m, mdgen.STREAM_B)
    Ag, Bg = torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda()
    T = torch.full((P, n, tile), 7.0, dtype=torch.float64, device="cuda")
    beta = torch.zeros((P, n), dtype=torch.float64, device="cuda")
    M.qr(P, Ag, tile, T=T, beta=beta)
    F, bt = Ag.cpu().numpy(), beta.cpu().numpy()
    ref = orc.apply_qt(F, bt, B)  # the library's own reflectors: no condition number enters
    M.apply_qt(P, Ag, T, Bg, tile)
    tol = 64 * m * unit(P)
    err = md_err(Bg.cpu().numpy(), ref)
    print("  Q^T B %.2f u" % (err / unit(P)), flush=True)
    assert err <= tol
    M.apply_q(P, Ag, T, Bg, tile)
    err = md_err(Bg.cpu().numpy(), B)
    print("  Q Q^T B %.2f u" % (err / unit(P)), flush=True)
    assert err <= 2 * tol
    Tn = T.cpu().numpy()
    for j in range(n):  # upper triangular, betas on the diagonal
        assert np.all(Tn[:, j, j % tile + 1:] == 0.0)
        assert np.array_equal(Tn[:, j, j % tile], bt[:, j])


# P, m, n, tile, columns of B: on both sides of where each of the three products changes form (a wave per output
# or 64 rows, a thread per row, blocks of outputs); more columns than one launch takes, the last launch with few
ROUTES = [
    (2, 300, 256, 256, 352), (2, 300, 256, 256, 400), (2, 290, 256, 128, 700), (2, 1100, 16, 16, 150), (2, 2000, 8, 8, 130),
    (2, 100, 60, 2, 40), (2, 100, 60, 4, 40), (2, 40, 33, 33, 3000),
    (4, 280, 256, 256, 180), (4, 280, 256, 256, 200), (4, 700, 48, 48, 100), (4, 1200, 32, 32, 64), (4, 600, 24, 8, 120),
    (4, 90, 40, 1, 30), (4, 150, 96, 96, 205), (4, 64, 64, 64, 590),
    (8, 260, 256, 256, 260), (8, 260, 256, 128, 130), (8, 200, 32, 16, 300), (8, 70, 20, 4, 20), (8, 60, 20, 1, 17),
    (1, 300, 256, 256, 400), (1, 300, 64, 32, 700),
]


@pytest.mark.parametrize("P,m,n,tile,nrhs", ROUTES)
def test_apply_form_of_the_products(P, m, n, tile, nrhs):
    """All columns in one call against the same columns nine at a time (each a wave per output, held to the
    oracle above): Q^T B and Q B agree to 64 m u whatever form the number of columns chooses, and Q Q^T B is B."""
    import paper_2110_08375_amd as M

    print("case apply form P=%d m=%d n=%d tile=%d nrhs=%d" % (P, m, n, tile, nrhs), flush=True)
    Ag = torch.from_numpy(mdgen.md_uniform(P, m, n, 510 + m, mdgen.STREAM_A)).cuda()
    B = mdgen.md_uniform(P, m, nrhs, 610 + m, mdgen.STREAM_B)
    Bg = torch.from_numpy(B).cuda()
    T = torch.full((P, n, tile), 7.0, dtype=torch.float64, device="cuda")
    M.qr(P, Ag, tile, T=T)
    tol = 64 * m * unit(P)
    for apply in (M.apply_qt, M.apply_q):
        few = Bg.clone()
        for c in range(0, nrhs, 9):
            part = few[:, c:c + 9].contiguous()
            apply(P, Ag, T, part, tile)
            few[:, c:c + 9] = part
        apply(P, Ag, T, Bg, tile)
        err = md_err(Bg.cpu().numpy(), few.cpu().numpy())
        print("  %.2f u" % (err / unit(P)), flush=True)
        assert err <= tol
    assert md_err(Bg.cpu().numpy(), B) <= 2 * tol


@pytest.mark.parametrize("P,m,n,tile,nrhs", [(2, 90, 64, 64, 3), (2, 300, 256, 256, 400), (4, 90, 64, 64, 3),
                                             (4, 300, 256, 256, 210), (8, 70, 48, 48, 3), (8, 270, 256, 256, 260),
                                             (4, 60, 8, 2, 20), (1, 300, 256, 256, 400)])
def test_apply_nan_column_leaves_the_rows_above(P, m, n, tile, nrhs):
    """A NaN in column j of A makes that reflector and those after it NaN: the first j rows of Q^T B do not
    depend on them and keep their bits, whatever form the products take."""
    import paper_2110_08375_amd as M

    print("case apply nan P=%d m=%d n=%d tile=%d nrhs=%d" % (P, m, n, tile, nrhs), flush=True)
    A = mdgen.md_uniform(P, m, n, 520 + m, mdgen.STREAM_A)
    Bg = torch.from_numpy(mdgen.md_uniform(P, m, nrhs, 620 + m, mdgen.STREAM_B)).cuda()
    T = torch.zeros((P, n, tile), dtype=torch.float64, device="cuda")
    Ag = torch.from_numpy(A).cuda()
    M.qr(P, Ag, tile, T=T)
    ref = M.apply_qt(P, Ag, T, Bg.clone(), tile)
    for j in (3, tile // 2 + 1, n - 2):
        An = A.copy()
        An[0, j, j + 1] = np.nan
        Ag = torch.from_numpy(An).cuda()
        M.qr(P, Ag, tile, T=T)
        out = M.apply_qt(P, Ag, T, Bg.clone(), tile)
        assert bool(torch.isnan(out[0, :, j:]).all()), j
        assert torch.equal(out[:, :, :j], ref[:, :, :j]), j
