"""GPU parity of the factorisation whose launches hold a panel and the previous panel's update side by
side, at the edges of its layout: rows around the 128 of a staged chunk, one more and one less than
where two waves share a column, the largest number of rows it takes and one more (the other form),
ragged last panels, few columns.  x, R and Q^T b against the oracle."""
import numpy as np
import pytest

import mdgen

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def unit(P):
    return 2.0 ** -(53 * P - (P - 1))


def md_diff(x, ref):
    d = np.zeros(ref.shape[1:])
    for k in range(ref.shape[0] - 1, -1, -1):
        d = d + (x[k] - ref[k])
    return np.max(np.abs(d)) / np.max(np.abs(ref[0]))


CASES = [
    # P, m, n
    (2, 127, 20), (2, 128, 128), (2, 129, 33), (2, 257, 49), (2, 1024, 36), (2, 1025, 36), (2, 17, 17), (2, 16, 1),
    (2, 4096, 18), (2, 4097, 18), (4, 129, 17), (4, 768, 20), (4, 769, 20), (4, 130, 130), (4, 9, 9), (4, 2048, 10),
    (4, 2049, 10), (1, 300, 70), (1, 1030, 40),
]


@pytest.mark.parametrize("P,m,n", CASES)
def test_step_edges(orc, P, m, n):
    import paper_2110_08375_amd as M

    print("case step P=%d m=%d n=%d" % (P, m, n), flush=True)
    A = mdgen.md_uniform(P, m, n, 700 + m, mdgen.STREAM_A)
    b = mdgen.md_vector(P, m, 701 + n, mdgen.STREAM_B)
    ref = orc.lstsq(A, b)
    Ag, bg = torch.from_numpy(A).cuda(), torch.from_numpy(b).cuda()
    x, info = M.solve(P, Ag, bg, 1)
    assert int(info.item()) == 0
    k = float(np.linalg.cond(A[0].T))
    tol = 64 * n * unit(P) * max(1.0, k)
    F = Ag.cpu().numpy()
    R = np.stack([np.triu(F[l].T[:n, :]) for l in range(P)])
    Ro = np.stack([np.triu(ref["F"][l].T[:n, :]) for l in range(P)])
    errs = (md_diff(x.cpu().numpy(), ref["x"]), md_diff(R, Ro), md_diff(bg.cpu().numpy(), ref["qtb"]))
    print("  x %.2f, R %.2f, Q^T b %.2f u kappa" % tuple(e / (unit(P) * k) for e in errs), flush=True)
    assert max(errs) <= tol


@pytest.mark.parametrize("P,m,n", [(2, 1100, 90), (4, 800, 40)])
def test_step_grid_cap_and_lookahead_keep_the_bits(P, m, n):
    """The update's grid cap (its workgroups then take several column groups each) and the look-ahead
    switch change no bit."""
    import paper_2110_08375_amd as M
    from paper_2110_08375_amd import mdls

    A = mdgen.md_uniform(P, m, n, 31, mdgen.STREAM_A)
    b = mdgen.md_vector(P, m, 32, mdgen.STREAM_B)
    out = []
    for opt, val in ((mdls.MDLS_TUNE_APPLY_GRID_CAP, 0), (mdls.MDLS_TUNE_APPLY_GRID_CAP, 3), (mdls.MDLS_TUNE_LOOKAHEAD, 0)):
        saved = M.get_tuning(opt)
        M.set_tuning(opt, val)
        try:
            Ag, bg = torch.from_numpy(A).cuda(), torch.from_numpy(b).cuda()
            x, _ = M.solve(P, Ag, bg, 10)
            out.append((x.cpu().numpy(), Ag.cpu().numpy(), bg.cpu().numpy()))
        finally:
            M.set_tuning(opt, saved)
    for o in out[1:]:
        assert all(np.array_equal(p, q) for p, q in zip(out[0], o))


@pytest.mark.parametrize("P,m,n,off", [(2, 300, 100, 0), (2, 300, 100, 100), (4, 200, 150, 0), (4, 64, 64, 0), (4, 90, 64, 7),
                                       (8, 80, 70, 0), (1, 300, 100, 0), (1, 300, 100, 30)])
def test_solution_over_the_right_hand_side(P, m, n, off):
    """x in b's own memory, at its start or further on, with m > n and m == n: the same bits as in
    memory of its own."""
    import paper_2110_08375_amd as M

    print("case x over b P=%d m=%d n=%d off=%d" % (P, m, n, off), flush=True)
    A = torch.from_numpy(mdgen.md_uniform(P, m, n, 5, mdgen.STREAM_A)).cuda()
    b = torch.from_numpy(mdgen.md_vector(P, m, 6, mdgen.STREAM_B)).cuda()
    ref, info = M.solve(P, A.clone(), b.clone(), 1)
    assert int(info.item()) == 0
    buf = torch.zeros(P * (m + n), dtype=torch.float64, device="cuda")
    for _ in range(3):
        bb, x = buf[:P * m].view(P, m), buf[off:off + P * n].view(P, n)
        bb.copy_(b)
        _, info = M.solve(P, A.clone(), bb, 1, x=x)
        assert int(info.item()) == 0
        assert torch.equal(x, ref)


@pytest.mark.parametrize("P,m,n", [(4, 128, 5), (4, 129, 5), (4, 137, 12), (2, 512, 9), (2, 513, 9), (2, 545, 35), (1, 1024, 7),
                                   (1, 1025, 7), (2, 600, 1)])
def test_step_tail_edges(orc, P, m, n):
    """The last panel's update of the right-hand side alone, at the rows from which it is cut up."""
    test_step_edges(orc, P, m, n)
