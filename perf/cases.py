"""Cases that time the library through its public calls.

Each case is one call (or the short sequence of calls that belongs together) of the binding in
``paper_2110_08375_amd``: the plain least-squares solve in double double, quad double and octo
double from the smallest square system to the tall one, the back substitution alone at the size
the paper reports, a batch of uneven problems, the refined solve, the complex solve, and the QR
with the explicit orthogonal factor.  Entries are uniform in [-1, 1) with lower limbs uniform
below half an ulp of the limb above, the recipe of the benchmark and the tests.

The calls overwrite A and b in place, so a pass first restores them from the pristine copies that
a program solving the same system again would also keep.
"""
import math

import numpy as np
import torch

import paper_2110_08375_amd as mdls

# md multiply-add in FP64 instructions of an FMA machine when products are formed with an FMA and
# sums with TwoSum; used only to state the least work of a case in plain FP64 operations
FMA_FLOPS = {2: 15.0, 4: 125.0, 8: 1000.0}


# ------------------------------------------------------------------------------ the cases
def listed():
    return [
        # the smallest real use: one small square system (the smoke test's), where launches and
        # the latency of each column count
        {"name": "solve dd 128", "kind": "solve", "p": 2, "m": 128, "n": 128, "tile": 32},
        # an ordinary data-fitting size, taller than wide, no power of two anywhere
        {"name": "solve qd 500x300", "kind": "solve", "p": 4, "m": 500, "n": 300, "tile": 60},
        # the benchmark's three solves (the paper's least-squares table)
        {"name": "solve dd 1024", "kind": "solve", "p": 2, "m": 1024, "n": 1024, "tile": 128},
        {"name": "solve qd 1024", "kind": "solve", "p": 4, "m": 1024, "n": 1024, "tile": 128},
        {"name": "solve od 1024", "kind": "solve", "p": 8, "m": 1024, "n": 1024, "tile": 128},
        # overdetermined, in the highest precision: twice the rows
        {"name": "solve od 2048x1024", "kind": "solve", "p": 8, "m": 2048, "n": 1024, "tile": 128},
        # the tiled back substitution alone, at the size of the paper's table
        {"name": "backsub qd 17920", "kind": "backsub", "p": 4, "m": 17920, "n": 17920, "tile": 256},
        # many independent uneven problems in one launch, as a path tracker hands them over
        {"name": "batch dd 512", "kind": "batch", "p": 2, "m": 512, "n": 512, "count": 512},
        {"name": "batch qd 160", "kind": "batch", "p": 4, "m": 512, "n": 512, "count": 160},
        # octo-double accuracy from a double-double factorisation, kappa = 1e8
        {"name": "refined od 2048", "kind": "refined", "p": 8, "m": 2048, "n": 2048, "tile": 128},
        # the paper's complex workload, solved
        {"name": "csolve dd 512", "kind": "csolve", "p": 2, "m": 512, "n": 512, "tile": 128},
        # QR with the tile factors, then the explicit orthogonal matrix, as the paper's QR forms it
        {"name": "qr+q qd 1024", "kind": "form_q", "p": 4, "m": 1024, "n": 1024, "tile": 128},
    ]


def _size(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["solve", "solve", "solve", "solve", "solve", "backsub", "batch", "batch", "refined", "csolve",
                       "form_q"])
    if kind == "batch":
        # m the largest number of rows
        p, m = rng.choice([2, 4]), rng.randint(64, 512)
        return {"kind": kind, "p": p, "m": m, "n": m, "count": _size(rng, 16, 512 if p == 2 else 160)}
    if kind == "backsub":
        p, tile = rng.choice([2, 4, 8]), rng.choice([32, 48, 64, 96, 128, 256])
        n = tile * max(1, _size(rng, 256, {2: 17920, 4: 17920, 8: 6000}[p]) // tile)
        return {"kind": kind, "p": p, "m": n, "n": n, "tile": tile}
    if kind == "refined":
        p, tile = rng.choice([4, 8]), rng.choice([32, 64, 128])
        n = tile * max(1, _size(rng, 128, 2048) // tile)
        return {"kind": kind, "p": p, "m": n if rng.random() < 0.5 else rng.randint(n, min(2048, 2 * n)), "n": n,
                "tile": tile}
    p = rng.choice([2, 4, 8] if kind != "csolve" else [2, 2, 4])
    top = {"solve": 1024, "csolve": 512, "form_q": {2: 1024, 4: 1024, 8: 640}[p]}[kind]
    tile = rng.choice([8, 20, 32, 48, 64, 100, 128])
    n = tile * max(1, _size(rng, 32, top) // tile)
    m = n if rng.random() < 0.5 else rng.randint(n, min(2 * n, 2048 if kind == "solve" else 1024))
    return {"kind": kind, "p": p, "m": m, "n": n, "tile": tile}


# ------------------------------------------------------------------------------ inputs
def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _uniform(shape, g):
    return torch.rand(shape, generator=g, dtype=torch.float64, device="cuda").mul_(2.0).sub_(1.0)


def _limbs(lead, p, g):
    """Lower limbs below half an ulp of the limb above; shape (p,) + lead.shape."""
    out = torch.empty((p,) + tuple(lead.shape), dtype=torch.float64, device="cuda")
    out[0] = lead
    for k in range(1, p):
        e = torch.frexp(out[k - 1]).exponent
        out[k] = torch.ldexp(_uniform(lead.shape, g), e - 54)
    return out


def _batch_shapes(case, seed):
    r = np.random.default_rng(int(seed))
    m = r.integers(32, case["m"] + 1, case["count"])
    n = r.integers(16, m + 1)
    return [(int(a), int(b)) for a, b in zip(m, n)]


def _inputs(case, seed):
    kind, p, m, n = case["kind"], case["p"], case["m"], case["n"]
    g = _gen(seed)
    if kind == "batch":
        shapes = _batch_shapes(case, 1)  # the same shapes for every seed: one plan serves them all
        descs, la, lb, _ = mdls.batch_descs(p, shapes)
        A = torch.empty(la, dtype=torch.float64, device="cuda")
        b = torch.empty(lb, dtype=torch.float64, device="cuda")
        a0 = sum(s[0] * s[1] for s in shapes)
        b0 = sum(s[0] for s in shapes)
        allA, allb = _limbs(_uniform((a0,), g), p, g), _limbs(_uniform((b0,), g), p, g)
        ia = ib = 0
        for d, (mm, nn) in zip(descs, shapes):
            A[d.a_off:d.a_off + p * mm * nn].view(p, mm * nn).copy_(allA[:, ia:ia + mm * nn])
            b[d.b_off:d.b_off + p * mm].view(p, mm).copy_(allb[:, ib:ib + mm])
            ia, ib = ia + mm * nn, ib + mm
        return A, b
    if kind == "backsub":
        # diagonal in [1, 2], the rows above it scaled so that the triangle is well conditioned
        lead = _uniform((n, n), g)
        i = torch.arange(n, device="cuda")
        lead.mul_(2.0 ** -math.ceil(math.log2(n))).mul_(i[None, :] < i[:, None])
        lead[i, i] = 1.5 + 0.5 * _uniform((n,), g)
        return _limbs(lead, p, g), _limbs(_uniform((n,), g), p, g)
    if kind == "refined":
        # U diag(s) V^T with s log-spaced down to 1e-8, U and V products of reflectors
        lead = torch.zeros((n, m), dtype=torch.float64, device="cuda")  # [column, row]
        i = torch.arange(n, device="cuda")
        lead[i, i] = torch.logspace(0.0, -8.0, n, dtype=torch.float64, device="cuda")
        for _ in range(8):
            u, v = _uniform((m,), g), _uniform((n,), g)
            lead.sub_(torch.outer(lead @ u, u * (2.0 / (u @ u))))
            lead.sub_(torch.outer(v * (2.0 / (v @ v)), v @ lead))
        return _limbs(lead, 2, g), _limbs(_uniform((m,), g), p, g)
    if kind == "csolve":
        A = torch.stack([_limbs(_uniform((n, m), g), p, g) for _ in range(2)])
        return A, torch.stack([_limbs(_uniform((m,), g), p, g) for _ in range(2)])
    return _limbs(_uniform((n, m), g), p, g), _limbs(_uniform((m,), g), p, g)


# ------------------------------------------------------------------------------ one pass
def prepare(case, seed):
    kind, p, m, n, tile = (case.get(k) for k in ("kind", "p", "m", "n", "tile"))
    A0, b0 = _inputs(case, seed)
    mdls.init()
    new = lambda *shape: torch.empty(shape, dtype=torch.float64, device="cuda")
    s = {"case": case, "A0": A0, "b0": b0, "info": torch.zeros(1, dtype=torch.int32, device="cuda")}
    if kind in ("solve", "csolve"):
        lead = (2,) if kind == "csolve" else ()
        ws = mdls.cworkspace if kind == "csolve" else mdls.workspace
        s.update(A=torch.empty_like(A0), b=torch.empty_like(b0), x=new(*lead, p, n), ws=ws(p, m, n, tile))
    elif kind == "backsub":
        s.update(x=torch.empty_like(b0), ws=mdls.workspace(p, n, n, tile))
    elif kind == "batch":
        descs, _, _, lx = mdls.batch_descs(p, _batch_shapes(case, 1))
        ws = mdls.batch_workspace(p, case["count"])
        mdls.batch_plan(p, descs, ws)
        s.update(A=torch.empty_like(A0), b=torch.empty_like(b0), x=new(lx), ws=ws,
                 info=torch.zeros(case["count"], dtype=torch.int32, device="cuda"),
                 variant=1)  # the autotuner's choice for such batches in both precisions
    elif kind == "refined":
        s.update(F=torch.empty_like(A0), x=new(p, n), ws=mdls.refined_workspace(p, m, n, tile), iters=10,
                 norms=torch.zeros(20, dtype=torch.float64, device="cuda"))
    else:
        s.update(A=torch.empty_like(A0), T=new(p, n, tile), Q=new(p, m, m), beta=new(p, n),
                 ws=mdls.workspace(p, m, n, tile))
    return s


def run(s):
    case = s["case"]
    kind, p, tile = case["kind"], case["p"], case.get("tile")
    if kind == "backsub":
        s["x"].copy_(s["b0"])
        x, info = mdls.backsub(p, s["A0"], s["x"], tile, ws=s["ws"], info=s["info"])
        return {"x": x, "info": info}
    if kind == "refined":
        x, info, _ = mdls.solve_refined(p, s["A0"], s["b0"], tile, s["iters"], x=s["x"], F=s["F"], ws=s["ws"],
                                        info=s["info"], norms=s["norms"])
        return {"x": x, "info": info, "factors": s["F"]}
    s["A"].copy_(s["A0"])
    if kind == "form_q":
        mdls.qr(p, s["A"], tile, T=s["T"], ws=s["ws"], beta=s["beta"], info=s["info"])
        mdls.form_q(p, s["A"], s["T"], tile, s["Q"], ws=s["ws"])
        return {"factors": s["A"], "T": s["T"], "beta": s["beta"], "Q": s["Q"], "info": s["info"]}
    s["b"].copy_(s["b0"])
    if kind == "batch":
        mdls.solve_batched(p, case["count"], s["A"], s["b"], s["x"], s["variant"], s["ws"], s["info"])
        return {"x": s["x"], "info": s["info"], "factors": s["A"], "qtb": s["b"]}
    solve = mdls.csolve if kind == "csolve" else mdls.solve
    x, info = solve(p, s["A"], s["b"], tile, x=s["x"], ws=s["ws"], info=s["info"])
    return {"x": x, "info": info, "factors": s["A"], "qtb": s["b"]}


# ------------------------------------------------------------------------------ least work
def _qr_fmas(m, n):
    return m * n * n - n ** 3 / 3.0


def work(case):
    kind, p, m, n = case["kind"], case["p"], case["m"], case["n"]
    if kind == "batch":
        shapes = _batch_shapes(case, 1)
        fmas = sum(_qr_fmas(a, b) + 2.0 * a * b + b * b / 2.0 for a, b in shapes)
        words = sum(2.0 * a * b + 2.0 * a + b for a, b in shapes) * p
    elif kind == "backsub":
        fmas, words = n * n / 2.0, p * (n * n / 2.0 + 2.0 * n)
    elif kind == "refined":
        # the factorisation in double double; residuals and solves are lower-order
        fmas, words, p = _qr_fmas(m, n), 2 * 2.0 * m * n + p * (m + n), 2
    elif kind == "csolve":
        fmas, words = 4.0 * (_qr_fmas(m, n) + 2.0 * m * n + n * n / 2.0), 2.0 * p * (2.0 * m * n + 2.0 * m + n)
    elif kind == "form_q":
        fmas, words = _qr_fmas(m, n) + 2.0 * m * m * n - m * n * n, p * (2.0 * m * n + m * m)
    else:
        fmas, words = _qr_fmas(m, n) + 2.0 * m * n + n * n / 2.0, p * (2.0 * m * n + 2.0 * m + n)
    return {"bytes": 8.0 * words, "flops": FMA_FLOPS[p] * fmas}


# ------------------------------------------------------------------------------ in 64 bits
def _lstsq(A, b):
    """A [column, row]; x in the leading limb's precision"""
    q, r = np.linalg.qr(A.T)
    y = q.conj().T @ b
    return np.linalg.solve(r, y)


def _planes(x, p):
    out = np.zeros((p,) + x.shape)
    out[0] = x
    return out


def exact(case, seed):
    kind, p, n = case["kind"], case["p"], case["n"]
    A, b = _inputs(case, seed)
    if kind == "batch":
        shapes = _batch_shapes(case, 1)
        descs, _, _, lx = mdls.batch_descs(p, shapes)
        Ah, bh, x = A.cpu().numpy(), b.cpu().numpy(), np.zeros(lx)
        for d, (mm, nn) in zip(descs, shapes):
            x[d.x_off:d.x_off + nn] = _lstsq(Ah[d.a_off:d.a_off + mm * nn].reshape(nn, mm), bh[d.b_off:d.b_off + mm])
        return {"x": x, "info": None, "factors": None, "qtb": None}
    if kind == "backsub":
        x = torch.linalg.solve_triangular(A[0].T, b[0][:, None], upper=True)[:, 0]
        return {"x": _planes(x.cpu().numpy(), p), "info": None}
    if kind == "csolve":
        x = _lstsq((A[0, 0] + 1j * A[1, 0]).cpu().numpy(), (b[0, 0] + 1j * b[1, 0]).cpu().numpy())
        return {"x": np.stack([_planes(x.real, p), _planes(x.imag, p)]), "info": None, "factors": None, "qtb": None}
    if kind == "form_q":
        q, r = np.linalg.qr(A[0].cpu().numpy().T, mode="complete")
        if case["m"] > n:  # the columns past n are any basis of the complement
            return {"factors": None, "T": None, "beta": None, "Q": None, "info": None}
        q = q * np.where(np.diagonal(r) < 0.0, -1.0, 1.0)  # R has a non-negative diagonal
        if np.linalg.slogdet(q)[0] != (-1.0) ** (n - 1):  # n - 1 reflectors: none acts on the last row
            q[:, n - 1] *= -1.0
        return {"factors": None, "T": None, "beta": None, "Q": _planes(q.T, p), "info": None}
    if kind == "refined" and case["m"] > n:  # kappa^2 times a residual: nothing left of it in 64 bits
        return None
    x = _lstsq(A[0].cpu().numpy(), b[0].cpu().numpy())
    res = {"x": _planes(x, p), "info": None, "factors": None}
    return res if kind == "refined" else {**res, "qtb": None}
