"""GPU parity of the one-launch back substitution at the edges of its layout: fewer rows than a block
of 32, one more and one less than a block, an odd number of blocks, around the number of blocks from
which it works ahead of the chain (22), a leading dimension larger than n."""
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


def problem(P, n, ldr):
    R = np.full((P, n, ldr), np.nan)  # what lies below the diagonal is not read
    U = mdgen.upper_triangular(P, n, 40 + n, well_conditioned=True)
    for c in range(n):
        R[:, c, :c + 1] = U[:, c, :c + 1]
    return U, R, mdgen.md_vector(P, n, 41, mdgen.STREAM_B)


SIZES = [(1, 1), (5, 5), (31, 31), (32, 40), (33, 33), (64, 64), (65, 65), (96, 97), (703, 703), (704, 704), (705, 710),
         (737, 737)]


@pytest.mark.parametrize("P", (1, 2, 4))
@pytest.mark.parametrize("n,ldr", SIZES)
def test_trsv_edges(orc, P, n, ldr):
    check(orc, P, n, ldr)


@pytest.mark.parametrize("n,ldr", [(1, 1), (33, 33), (64, 70), (90, 90), (736, 736)])
def test_trsv_edges_od(orc, n, ldr):
    check(orc, 8, n, ldr)


def check(orc, P, n, ldr):
    import paper_2110_08375_amd as M

    print("case trsv P=%d n=%d ldr=%d" % (P, n, ldr), flush=True)
    U, R, y = problem(P, n, ldr)
    x, info = M.backsub(P, torch.from_numpy(R).cuda(), torch.from_numpy(y).cuda(), 1)
    assert int(info.item()) == 0
    ref, _ = orc.backsub(U, y)
    k = float(np.linalg.cond(U[0].T))
    err = md_err(x.cpu().numpy(), ref)
    print("  %.2f u kappa" % (err / (unit(P) * k)), flush=True)
    assert err <= 64 * n * unit(P) * max(1.0, k)


def test_trsv_status():
    """A zero diagonal entry is reported (the first one), and a wait that gives up at once ends with -1."""
    import paper_2110_08375_amd as M
    from paper_2110_08375_amd import mdls

    U, _, y = problem(2, 150, 150)
    U[:, 120, 120] = 0.0
    U[:, 77, 77] = 0.0
    _, info = M.backsub(2, torch.from_numpy(U).cuda(), torch.from_numpy(y).cuda(), 1)
    assert int(info.item()) == 78
    U, _, y = problem(2, 1500, 1500)
    Ug = torch.from_numpy(U).cuda()
    saved = M.get_tuning(mdls.MDLS_TUNE_SPIN_LIMIT)
    M.set_tuning(mdls.MDLS_TUNE_SPIN_LIMIT, 0)
    try:
        _, info = M.backsub(2, Ug, torch.from_numpy(y).cuda(), 1)
        assert int(info.item()) == -1
    finally:
        M.set_tuning(mdls.MDLS_TUNE_SPIN_LIMIT, saved)
    _, info = M.backsub(2, Ug, torch.from_numpy(y).cuda(), 1)
    assert int(info.item()) == 0


@pytest.mark.parametrize("P,n", [(1, 1500), (2, 200), (2, 1500), (4, 900), (8, 1100)])
def test_trsv_status_of_a_wait_that_gave_up(P, n):
    """With a spin limit of 0 or 2 polls waits give up or not as the workgroups happen to run: x is then
    either the solution or *info is -1, in each of ten runs."""
    import paper_2110_08375_amd as M
    from paper_2110_08375_amd import mdls

    print("case trsv status P=%d n=%d" % (P, n), flush=True)
    U, _, y = problem(P, n, n)
    Ug, yg = torch.from_numpy(U).cuda(), torch.from_numpy(y).cuda()
    ref, info = M.backsub(P, Ug, yg.clone(), 1)
    assert int(info.item()) == 0
    saved = M.get_tuning(mdls.MDLS_TUNE_SPIN_LIMIT)
    try:
        for rep in range(10):
            M.set_tuning(mdls.MDLS_TUNE_SPIN_LIMIT, 2 * (rep % 2))
            x, info = M.backsub(P, Ug, yg.clone(), 1)
            assert int(info.item()) in (0, -1)
            assert int(info.item()) == -1 or torch.equal(x, ref), rep
    finally:
        M.set_tuning(mdls.MDLS_TUNE_SPIN_LIMIT, saved)


@pytest.mark.parametrize("bad", (np.nan, np.inf))
@pytest.mark.parametrize("P,n", [(1, 90), (2, 90), (4, 90), (8, 70), (1, 800), (2, 800), (4, 800), (8, 1184)])
def test_trsv_nan_and_inf_stay_above(P, n, bad):
    """A NaN or Inf in y(r), in R(r, r) or in R(r, c) reaches x(0:r+1) and leaves every x below row r as it
    is, bit for bit, wherever r lies in a block of rows."""
    import paper_2110_08375_amd as M

    print("case trsv nan P=%d n=%d %s" % (P, n, bad), flush=True)
    U, _, y = problem(P, n, n)
    Ug, yg = torch.from_numpy(U).cuda(), torch.from_numpy(y).cuda()
    ref, _ = M.backsub(P, Ug, yg.clone(), 1)
    assert bool(torch.isfinite(ref).all())
    for r in (0, 5, 18, 31, 32, 50, n - 2):
        yb = yg.clone()
        yb[0, r] = bad
        x, _ = M.backsub(P, Ug, yb, 1)
        assert torch.equal(x[:, r + 1:], ref[:, r + 1:]), ("y", r)
        assert not bool(torch.isfinite(x[0, r])), ("y", r)
        for c in (r, r + 1, min(n - 1, r + 32), n - 1):
            Ub = Ug.clone()
            Ub[0, c, r] = bad
            x, _ = M.backsub(P, Ub, yg.clone(), 1)
            assert torch.equal(x[:, r + 1:], ref[:, r + 1:]), ("R", r, c)
            assert np.isinf(bad) and r == c or not bool(torch.isfinite(x[0, r])), ("R", r, c)


# on both sides of where the caller's tiles take over from the one launch, and where that works ahead of the chain
TILES = [
    (4, 8, 8), (4, 24, 8), (4, 32, 8), (4, 48, 24), (4, 64, 32), (4, 96, 32), (4, 64, 64), (4, 1, 1), (4, 2, 1),
    (8, 1, 1), (8, 4, 2), (8, 32, 4), (8, 64, 8), (8, 72, 8), (8, 120, 20), (8, 31, 31), (8, 96, 32), (8, 96, 48), (8, 100, 50),
    (8, 192, 64), (8, 256, 64), (8, 832, 32), (8, 864, 32), (8, 896, 128), (8, 1024, 128), (8, 576, 96), (8, 1280, 4),
    (8, 1284, 4),
]


@pytest.mark.parametrize("P,n,tile", TILES)
def test_backsub_form_by_tile(orc, P, n, tile):
    import paper_2110_08375_amd as M

    print("case backsub form P=%d n=%d tile=%d" % (P, n, tile), flush=True)
    U, R, y = problem(P, n, n)
    x, info = M.backsub(P, torch.from_numpy(R).cuda(), torch.from_numpy(y).cuda(), tile)
    assert int(info.item()) == 0
    ref, _ = orc.backsub(U, y)
    k = float(np.linalg.cond(U[0].T))
    err = md_err(x.cpu().numpy(), ref)
    print("  %.2f u kappa" % (err / (unit(P) * k)), flush=True)
    assert err <= 64 * n * unit(P) * max(1.0, k)


@pytest.mark.parametrize("P,n,tile", [(8, 128, 16), (8, 1024, 128), (4, 32, 32)])
def test_solve_by_tiles_reports(P, n, tile):
    """Where the solve's back substitution goes by tiles: a zero column and a time-out of the factorisation
    are reported as before."""
    import paper_2110_08375_amd as M
    from paper_2110_08375_amd import mdls

    print("case solve by tiles P=%d n=%d" % (P, n), flush=True)
    A = torch.from_numpy(mdgen.md_uniform(P, n, n, 9, mdgen.STREAM_A)).cuda()
    b = torch.from_numpy(mdgen.md_vector(P, n, 9, mdgen.STREAM_B)).cuda()
    Az = A.clone()
    Az[:, n // 2, :] = 0.0
    _, info = M.solve(P, Az, b.clone(), tile)
    assert int(info.item()) == n // 2 + 1
    saved = M.get_tuning(mdls.MDLS_TUNE_SPIN_LIMIT)
    M.set_tuning(mdls.MDLS_TUNE_SPIN_LIMIT, 0)
    try:
        _, info = M.solve(P, A.clone(), b.clone(), tile)
        assert int(info.item()) == (-1 if n > 64 else 0)
    finally:
        M.set_tuning(mdls.MDLS_TUNE_SPIN_LIMIT, saved)
    _, info = M.solve(P, A.clone(), b.clone(), tile)
    assert int(info.item()) == 0
