"""Workloads of the framework, one dict of plain values each, and how to run them.

A workload is a random-feature-method (RFM) least-squares system min ||A x - b||
for the Poisson or Helmholtz problem on the unit square or cube (the systems of
rfmgen, built here on the GPU) and one call a program makes with it: the whole
pipeline (sketch, preconditioner, LSQR), a solve with a preconditioner the
program kept, the gradients, or the setup stages alone.

Keys of a case
  kind    solve     csqrp_lsqr on a new system (Alg. 1)
          svd       cssvdp_lsqr on a new system (Alg. 2)
          kept      rfmls_solve with A^T and the preconditioner kept: time steps,
                    parameter studies, more load cases for the same geometry
          backward  rfmls_solve_backward after a kept solve
          train     LstsqFunction forward and backward: a training step through
                    the solver, the values of A and b both differentiable
          setup     rfmls_transpose and rfmls_sketch (with S b)
  d, N, J, Q        dimension, boxes per axis, features per box, points per axis
  pde               poisson or helmholtz (d = 3)
  gamma             sketch rows per column
  nrhs              right-hand sides
  qr, store         precision of the factorisation and of the stored preconditioner
  start, refine, operator   options of the solve
  scale             feature weights and offsets are uniform in [-scale, scale]

scale is 1 in two dimensions, rfmgen's own choice.  Those systems have condition
numbers of 1e6 to 1e13, so their coefficients are not determined to any useful
accuracy and what a program takes from them is the solution field; the pass ends
with it, u_h at P points of every box.  In three dimensions scale is 3 (steeper
features, condition numbers of 1e3 to 1e5), the coefficients and residuals are
determined to about 1e-12, and the pass returns them, and the gradients, whole.
"""

import itertools
import math

import torch

import paper_2409_15818_amd as R

POINTS = {2: 8, 3: 4}  # points per axis and box at which a field is returned


def _case(name, kind, d, N, J, Q, **kw):
    c = dict(name=name, kind=kind, d=d, N=N, J=J, Q=Q, pde="poisson", gamma=4, nrhs=1, qr="f64", store="f64",
             start="zero", refine=1, operator="implicit", scale=1.0 if d == 2 else 3.0)
    c.update(kw)
    return c


def listed():
    return [
        # the smallest system a user starts with (the quick-start and smoke
        # size, n = 200): launches and host latency are most of it
        _case("solve_2d_2x2", "solve", 2, 2, 50, 20),
        # a medium 2D system (n = 1,600) with the sketched start
        _case("solve_2d_4x4", "solve", 2, 4, 100, 24, start="sketch", refine=2),
        # the 3D Helmholtz problem on 2^3 boxes (n = 3,200, m = 83,200): a tall
        # system with few columns
        _case("solve_helmholtz_2x2x2", "solve", 3, 2, 400, 20, pde="helmholtz", start="sketch", refine=2),
        # the headline system of the benchmark (n = 12,800, m = 112,640)
        _case("solve_2d_8x8", "solve", 2, 8, 200, 40, start="sketch", refine=2),
        # the widest system (n = 25,600, m = 165,888) with the float32
        # factorisation and stored inverse
        _case("solve_3d_4x4x4_f32", "solve", 3, 4, 400, 12, gamma=2, qr="f32", store="f32", start="sketch",
              refine=2),
        # Alg. 1 step 4 taken literally: B = A R^{-1} formed, odd sizes (n = 2,619)
        _case("solve_3d_explicit_odd", "solve", 3, 3, 97, 9, operator="explicit"),
        # the SVD preconditioner on the Helmholtz problem (n = 1,600)
        _case("svd_helmholtz_2x2x2", "svd", 3, 2, 200, 14, pde="helmholtz"),
        # one more right-hand side for a kept headline system (a time step)
        _case("kept_2d_8x8_1rhs", "kept", 2, 8, 200, 40, refine=2),
        # 32 load cases of a kept Helmholtz system, in lockstep
        _case("kept_helmholtz_32rhs", "kept", 3, 2, 400, 20, pde="helmholtz", nrhs=32),
        # gradients of a few load cases, odd sizes (n = 1,864, 7 right-hand sides)
        _case("backward_3d_7rhs_odd", "backward", 3, 2, 233, 13, nrhs=7),
        # a training step through a small solver (n = 720)
        _case("train_3d_2x2x2", "train", 3, 2, 90, 8, gamma=2),
        # transpose and float32 sketch of a large system (setup of many solves)
        _case("setup_3d_3x3x3_f32", "setup", 3, 3, 350, 14, gamma=2, qr="f32", nrhs=2),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["solve", "solve", "solve", "svd", "kept", "kept", "backward", "train", "setup"])
    d = 3 if kind in ("svd", "backward", "train") or rng.random() < 0.6 else 2
    nmax = {"svd": 1600, "train": 2400, "backward": 3200}.get(kind, 8000)
    N = rng.choice([2, 3, 4] if d == 3 else [2, 3, 4, 5, 6, 8])
    boxes = N ** d
    J = _log_int(rng, 24, max(32, min(400 if d == 3 else 200, nmax // boxes)))
    # points per axis: 2 to 8 interior points per feature
    Q = max(5, int(math.ceil((J * rng.uniform(2.0, 8.0)) ** (1.0 / d))))
    kw = dict(refine=2) if d == 2 else dict(gamma=rng.choice([2, 3, 4]))
    if d == 3 and rng.random() < 0.4:
        kw["pde"] = "helmholtz"
    if kind in ("solve", "kept") and d == 3 and rng.random() < 0.4:
        kw["qr"] = kw["store"] = "f32"
    if kind == "svd" and rng.random() < 0.3:
        kw["store"] = "f32"
    if kind == "solve":
        kw["start"] = rng.choice(["zero", "sketch"])
        kw["refine"] = kw.get("refine") or rng.choice([1, 2])
        kw["nrhs"] = rng.choice([1, 1, 1, _log_int(rng, 2, 40)])
        if rng.random() < 0.2 and boxes * J <= 4000:
            kw["operator"] = "explicit"
    elif kind in ("kept", "backward", "setup"):
        kw["nrhs"] = rng.choice([1, _log_int(rng, 2, 64 if kind == "kept" else 32)])
    if kind == "setup":
        kw["qr"] = rng.choice(["f64", "f32"])
    c = _case("", kind, d, N, J, Q, **kw)
    del c["name"]
    return c


# ---------------------------------------------------------------------------
# systems (rfmgen's construction, on the GPU)
# ---------------------------------------------------------------------------
def _grid(d, Q):
    """Q cell-centred points per axis of the box [-1, 1]^d, row-major: [Q^d, d]."""
    ax = (torch.arange(Q, dtype=torch.float64, device="cuda") + 0.5) * (2.0 / Q) - 1.0
    if d == 0:
        return torch.zeros((1, 0), dtype=torch.float64, device="cuda")
    return torch.cartesian_prod(*[ax] * d).reshape(-1, d)


def _features(z, W, B0):
    """tanh(w . z + b) of every box: z [boxes or 1, P, d] local points -> [boxes, P, J]."""
    t = B0[:, None, :].expand(-1, z.shape[1], -1).clone()
    for a in range(W.shape[2]):
        t += z[..., a:a + 1] * W[:, None, :, a]
    return torch.tanh_(t)


def _shape(c):
    """(m, n, nnz) of the system."""
    d, N, J, Q = c["d"], c["N"], c["J"], c["Q"]
    nb, face = N ** d, Q ** (d - 1)
    one = nb * Q ** d + 2 * d * N ** (d - 1) * face
    two = 2 * d * (N - 1) * N ** (d - 1) * face
    return one + two, nb * J, one * J + two * 2 * J


def _rhs(c, pts, k, shift):
    """The right-hand side f and the solution u of load case k at the points [.., d]."""
    d = c["d"]
    if c["pde"] == "helmholtz":
        ph = 2.0 * math.pi / 5.0 + shift
        x, y, z = (math.pi * pts[..., a] for a in range(3))
        ua = -torch.cos(x + ph) * torch.cos(y + ph) * torch.cos(z + ph)
        ub = -torch.cos(x + ph) * torch.cos(2 * y + ph) * torch.cos(4 * z + ph)
        a, b = 1.0 / k, 1.0 - 1.0 / k
        return a * (0.25 - 3 * math.pi ** 2) * ua + b * (0.25 - 21 * math.pi ** 2) * ub, a * ua + b * ub
    u = torch.sin(k * math.pi * pts[..., 0] + shift)
    for a in range(1, d):
        u = u * torch.sin(math.pi * pts[..., a] + shift)
    return (k * k + d - 1) * math.pi ** 2 * u, u


def _system(c, seed):
    """(A, b [nrhs, m], W, B0): the collocation system and its features."""
    d, N, J, Q = c["d"], c["N"], c["J"], c["Q"]
    gen = torch.Generator(device="cuda").manual_seed(int(seed))
    nb, r = N ** d, 1.0 / (2 * N)
    draws = (2.0 * torch.rand((nb, J, d + 1), generator=gen, dtype=torch.float64, device="cuda") - 1.0) * c["scale"]
    shift = 0.3 * float(torch.rand((), generator=gen, dtype=torch.float64, device="cuda"))
    W, B0 = draws[..., :d].contiguous(), draws[..., d].contiguous()
    boxes = list(itertools.product(range(N), repeat=d))
    ids = {bx: q for q, bx in enumerate(boxes)}
    centres = torch.tensor([[(2 * a + 1) * r for a in bx] for bx in boxes], dtype=torch.float64, device="cuda")
    modes = range(1, c["nrhs"] + 1)
    feat = torch.arange(J, device="cuda", dtype=torch.int32)
    vals, cols, widths, rhs = [], [], [], []

    def add(v, col):
        vals.append(v.reshape(-1))
        cols.append(col.expand(v.shape).reshape(-1))
        widths.append(torch.full((v.numel() // v.shape[-1],), v.shape[-1], dtype=torch.int64, device="cuda"))

    z = _grid(d, Q)[None]
    t = _features(z, W, B0)
    lap = 2.0 * t * (1.0 - t * t) * ((W * W).sum(-1) / (r * r))[:, None, :]
    q = torch.arange(nb, device="cuda", dtype=torch.int32)
    add(0.25 * t - lap if c["pde"] == "helmholtz" else lap, (q[:, None] * J + feat)[:, None, :])
    pts = centres[:, None, :] + r * z
    rhs.append(torch.stack([_rhs(c, pts, k, shift)[0].reshape(-1) for k in modes]))
    face = _grid(d - 1, Q)

    def on_face(axis, side):
        return torch.cat([face[:, :axis], torch.full((face.shape[0], 1), float(side), dtype=torch.float64,
                                                     device="cuda"), face[:, axis:]], dim=1)[None]

    for axis in range(d):
        for side in (-1, 1):
            sel = [ids[bx] for bx in boxes if bx[axis] == (0 if side < 0 else N - 1)]
            zf = on_face(axis, side)
            add(_features(zf, W[sel], B0[sel]), (q[sel][:, None] * J + feat)[:, None, :])
            pts = centres[sel][:, None, :] + r * zf
            rhs.append(torch.stack([_rhs(c, pts, k, shift)[1].reshape(-1) for k in modes]))
    for axis in range(d):
        lo = [ids[bx] for bx in boxes if bx[axis] < N - 1]
        hi = [ids[bx[:axis] + (bx[axis] + 1,) + bx[axis + 1:]] for bx in boxes if bx[axis] < N - 1]
        tp = _features(on_face(axis, 1), W[lo], B0[lo])
        tq = _features(on_face(axis, -1), W[hi], B0[hi])
        c0 = torch.cat([tp, -tq], dim=-1)
        c1 = torch.cat([(1 - tp * tp) * (W[lo][:, None, :, axis] / r), -(1 - tq * tq) * (W[hi][:, None, :, axis] / r)],
                       dim=-1)
        both = torch.cat([q[lo][:, None] * J + feat, q[hi][:, None] * J + feat], dim=1)
        add(torch.stack([c0, c1], dim=2), both[:, None, None, :])
        rhs.append(torch.zeros((c["nrhs"], 2 * tp.shape[0] * tp.shape[1]), dtype=torch.float64, device="cuda"))
    width = torch.cat(widths)
    ptr = torch.zeros(width.numel() + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(width, 0, out=ptr[1:])
    A = R.CSR(width.numel(), nb * J, ptr, torch.cat(cols).contiguous(), torch.cat(vals).contiguous())
    return A, torch.cat(rhs, dim=1).contiguous(), W, B0


def _rows(c):
    return c["gamma"] * c["N"] ** c["d"] * c["J"]


def _cotangent(c, n, seed):
    gen = torch.Generator(device="cuda").manual_seed(int(seed) + 977)
    return torch.randn((c["nrhs"], n), generator=gen, dtype=torch.float64, device="cuda")


def prepare(c, seed):
    A, b, W, B0 = _system(c, seed)
    if c["nrhs"] == 1 and c["kind"] != "setup":
        b = b[0].contiguous()
    st = {"case": c, "A": A, "b": b, "h": R.Handle(device="cuda:0"), "s": _rows(c),
          "opts": R.default_opts(refine=c["refine"])}
    if c["d"] == 2:
        st["basis"] = _features(_grid(2, POINTS[2])[None], W, B0)  # [boxes, P, J]
    kind = c["kind"]
    if kind in ("kept", "backward"):
        st["AT"] = R.rfmls_transpose(st["h"], A)
        SA, _, _, _ = R.rfmls_sketch(st["h"], A, st["s"], 2, dtype=c["qr"])
        st["P"] = R.rfmls_precond(st["h"], SA, c["qr"], c["store"])
        del SA
    if kind in ("backward", "train"):
        g = _cotangent(c, A.n, seed)
        st["G"] = g[0].contiguous() if c["nrhs"] == 1 else g
    if kind == "backward":
        st["X"], st["Rres"], _, _ = R.rfmls_solve(st["h"], A, st["AT"], st["P"], b, st["opts"])
    if kind == "train":
        st["solver"] = R.LstsqSolver(st["h"], A.m, A.n, A.row_ptr, A.col, st["s"], opts=st["opts"])
        st["val"] = A.val.clone().requires_grad_(True)
        st["b"] = b.clone().requires_grad_(True)
    return st


def _answer(st, x, res):
    """Coefficients and residuals, or the solution field at the points of every box."""
    if "basis" not in st:
        return {"x": x, "residual": res}
    basis = st["basis"]
    xb = x.reshape(-1, basis.shape[0], basis.shape[2]).permute(1, 2, 0).contiguous()
    return {"u": torch.bmm(basis, xb)}


def run(st):
    c, h, A = st["case"], st["h"], st["A"]
    kind = c["kind"]
    if kind == "solve":
        r = R.csqrp_lsqr(h, A, st["b"], st["s"], 2, c["qr"], c["store"], st["opts"], start=c["start"],
                         operator=c["operator"])
        return _answer(st, r.x, r.residual)
    if kind == "svd":
        r = R.cssvdp_lsqr(h, A, st["b"], st["s"], 2, p_store=c["store"], opts=st["opts"])
        return _answer(st, r.x, r.residual)
    if kind == "kept":
        x, res, _, _ = R.rfmls_solve(h, A, st["AT"], st["P"], st["b"], st["opts"])
        return _answer(st, x, res)
    if kind == "backward":
        db, dval, _, _ = R.rfmls_solve_backward(h, A, st["AT"], st["P"], st["X"], st["Rres"], st["G"], st["opts"])
        return {"db": db, "dval": dval}
    if kind == "train":
        x = st["solver"](st["val"], st["b"])
        dval, db = torch.autograd.grad(x, (st["val"], st["b"]), st["G"])
        return {"x": x.detach(), "db": db, "dval": dval}
    T = R.rfmls_transpose(h, A)
    SA, hsh, sgn, Sb = R.rfmls_sketch(h, A, st["s"], 2, b=st["b"], dtype=c["qr"], want_maps=True)
    return {"at_ptr": T.row_ptr, "at_col": T.col, "at_val": T.val, "SA": SA, "hash": hsh, "sign": sgn, "Sb": Sb}


# Iterations of LSQR on a system preconditioned through a sketch of gamma n
# rows: its singular values lie in 1 +- gamma^{-1/2}, so an iteration gains a
# factor gamma^{1/2}; ten digits, once from zero.
def _iterations(c):
    return math.ceil(10.0 / math.log10(math.sqrt(c["gamma"])))


def work(c):
    m, n, nnz = _shape(c)
    s, k, kind = _rows(c), c["nrhs"], c["kind"]
    esz = 4 if c["qr"] == "f32" else 8
    xsz = 4 if c["store"] == "f32" else 8
    vec = 8.0 * k * (m + n)
    csr = 8.0 * nnz + 4.0 * nnz + 8.0 * (m + 1)
    if kind == "setup":
        return {"bytes": 2 * csr + 8.0 * (n + 1) + esz * float(s) * n + 8.0 * k * (m + s) + 5.0 * m,
                "flops": 2.0 * nnz + 2.0 * k * m}
    # one iteration: A and A^T against the block of vectors, the preconditioner twice
    tri = n * (n + 1.0) / 2 if kind != "svd" else float(n) * n
    it = _iterations(c)
    solve_b = csr + xsz * tri + 2 * vec
    solve_f = it * k * (4.0 * nnz + 4.0 * tri)
    # Householder QR of the sketch and the triangular inverse
    pre_f = 2.0 * n * n * (s - n / 3.0) + n ** 3 / 3.0
    if kind == "svd":
        pre_f += 12.0 * n ** 3
    if kind == "kept":
        return {"bytes": solve_b, "flops": solve_f}
    if kind == "backward":
        return {"bytes": solve_b + 8.0 * nnz + vec, "flops": solve_f + 4.0 * k * nnz}
    both = {"bytes": solve_b, "flops": pre_f + solve_f}
    if kind == "train":
        both = {"bytes": both["bytes"] + 8.0 * nnz + vec, "flops": both["flops"] + solve_f + 4.0 * k * nnz}
    return both


# ---------------------------------------------------------------------------
# the same quantities by dense float64 algebra
# ---------------------------------------------------------------------------
def _dense(A):
    D = torch.zeros((A.m, A.n), dtype=torch.float64, device="cuda")
    rows = torch.repeat_interleave(torch.arange(A.m, device="cuda"), A.row_ptr[1:] - A.row_ptr[:-1])
    D[rows, A.col.long()] = A.val
    return D, rows


def _solve(U, B, upper):
    """U^{-1} B on the host, whose triangular solve takes any size."""
    return torch.linalg.solve_triangular(U.cpu(), B.cpu(), upper=upper).cuda()


def _triangular(D):
    """R of the QR factorisation of D: Cholesky of the column-scaled Gram matrix, twice."""
    sc = D.norm(dim=0)
    U1 = torch.linalg.cholesky((D / sc).T @ (D / sc)).T.contiguous()
    Q = (D / sc) @ _solve(U1, torch.eye(D.shape[1], dtype=D.dtype), True)
    U2 = torch.linalg.cholesky(Q.T @ Q).T.contiguous()
    return (U2 @ U1) * sc


def _lstsq(D, U, B):
    """Columns of X minimising ||D X - B||, by corrected semi-normal equations."""
    X = torch.zeros((D.shape[1], B.shape[1]), dtype=torch.float64, device="cuda")
    for _ in range(4):
        X = X + _solve(U, _solve(U.T, D.T @ (B - D @ X), False), True)
    return X


def exact(c, seed):
    m, n, nnz = _shape(c)
    # the ill-conditioned 2D systems need an orthogonal factorisation, which
    # plain torch takes long for beyond a couple of thousand columns
    if c["kind"] == "setup":
        return None
    if (c["d"] == 2 and n > 2000) or float(m) * n > 1.2e9:
        return None
    A, b, W, B0 = _system(c, seed)
    D, rows = _dense(A)
    one = c["nrhs"] == 1
    if c["d"] == 2:
        Dh, bh = D.cpu(), b.T.contiguous().cpu()
        sc = Dh.norm(dim=0)
        Qh, Uh = torch.linalg.qr(Dh / sc)
        X = torch.zeros((n, b.shape[0]), dtype=torch.float64)
        for _ in range(3):
            X = X + torch.linalg.solve_triangular(Uh, Qh.T @ (bh - (Dh / sc) @ X), upper=True)
        x = (X / sc[:, None]).T.contiguous().cuda()
        basis = _features(_grid(2, POINTS[2])[None], W, B0)
        return {"u": torch.bmm(basis, x.reshape(-1, basis.shape[0], basis.shape[2]).permute(1, 2, 0).contiguous())}
    U = _triangular(D)
    X = _lstsq(D, U, b.T.contiguous())
    Res = b.T - D @ X
    x, res = X.T.contiguous(), Res.T.contiguous()
    out = {"x": x[0] if one else x, "residual": res[0] if one else res}
    if c["kind"] in ("backward", "train"):
        G = _cotangent(c, n, seed).T.contiguous()
        Wt = _solve(U, _solve(U.T, G, False), True)
        Lam = D @ Wt
        cl = A.col.long()
        dval = torch.zeros(A.nnz, dtype=torch.float64, device="cuda")
        for k in range(c["nrhs"]):
            dval += Res[rows, k] * Wt[cl, k] - Lam[rows, k] * X[cl, k]
        db = Lam.T.contiguous()
        out = {"x": out["x"], "db": db[0] if one else db, "dval": dval}
        if c["kind"] == "backward":
            del out["x"]
    return out
