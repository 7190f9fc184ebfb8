"""GPU parity of the octo double panel's scalars spread over the lanes of a wave, at the edges of their form:
sigma far below and far above x1^2, x1 of either sign and zero, against the oracle within 64 n u kappa, as the
full-size solves; and matrices scaled by powers of two over the exponents it takes (|x|^2 < 2^900).  A scaling
by 2^k is exact, so the scaled factor is the scaled result."""
import numpy as np
import pytest

import mdgen

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

P = 8
UNIT = 2.0 ** -(53 * P - (P - 1))


def md_diff(x, ref):
    d = np.zeros(ref.shape[1:])
    for k in range(ref.shape[0] - 1, -1, -1):
        d = d + (x[k] - ref[k])
    return np.max(np.abs(d)) / np.max(np.abs(ref[0]))


def matrix(m, n, seed, kind):
    A = mdgen.md_uniform(P, m, n, seed, mdgen.STREAM_A)
    i = np.arange(n)
    if kind in ("pos", "neg"):  # x1 dominates: sigma ~ 2^-12 x1^2 and less
        A = A * 2.0 ** -12
        A[:, i, i] = 0.0
        A[0, i, i] = (1.0 if kind == "pos" else -1.0) * (1.0 + i / 64.0)
    elif kind == "zero":  # x1 = 0 in the first column; mixed signs after it
        A[:, 0, 0] = 0.0
    elif kind == "large":  # sigma dominates
        A[:, i, i] = A[:, i, i] * 2.0 ** -40
    return A


def factor(A, b):
    import paper_2110_08375_amd as M

    Ag, bg = torch.from_numpy(A).cuda(), torch.from_numpy(b).cuda()
    x, info = M.solve(P, Ag, bg, 1)
    assert int(info.item()) == 0
    n = A.shape[1]
    F = Ag.cpu().numpy()
    return np.stack([np.triu(F[l].T[:n, :]) for l in range(P)]), x.cpu().numpy()


@pytest.mark.parametrize("kind", ["pos", "neg", "zero", "large", "plain"])
@pytest.mark.parametrize("m,n", [(40, 17), (9, 9)])
def test_lanes_signs_and_sizes(orc, m, n, kind):
    print("case lanes m=%d n=%d %s" % (m, n, kind), flush=True)
    A = matrix(m, n, 900 + m, kind)
    b = mdgen.md_vector(P, m, 901, mdgen.STREAM_B)
    ref = orc.lstsq(A, b)
    R, x = factor(A, b)
    Ro = np.stack([np.triu(ref["F"][l].T[:n, :]) for l in range(P)])
    tol = 64 * n * UNIT * max(1.0, float(np.linalg.cond(A[0].T)))
    assert md_diff(R, Ro) <= tol
    assert md_diff(x, ref["x"]) <= tol


@pytest.mark.parametrize("e", [1, 101, 430, 446, -1, -100])
def test_lanes_scaled(e):
    """Entries up to 1, 40 rows: |x|^2 < 2^(2 e + 6): inside for all of these.  Downwards the last limb (2^-424 of an entry) stays normal for e >= -100 and so do the
    products' errors; x scales by 2^-e."""
    m, n = 40, 17
    print("case lanes scaled e=%d" % e, flush=True)
    A = matrix(m, n, 940, "plain")
    b = mdgen.md_vector(P, m, 901, mdgen.STREAM_B)
    R0, x0 = factor(A, b)
    R, x = factor(np.ldexp(A, e), b)
    tol = 64 * n * UNIT * max(1.0, float(np.linalg.cond(A[0].T)))
    assert md_diff(np.ldexp(R, -e), R0) <= tol
    assert md_diff(np.ldexp(x, e), x0) <= tol
