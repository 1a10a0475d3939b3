"""Workloads of the library, as a user's program calls them.

The work this library does for its users falls into seven operations, all
through the public binding (paper_2508_04917_amd.ddilu):

  apply     z = M^{-1} r with the domain-decomposed ILU0 (FP64, FP32-factor or
            FP32 arithmetic, with or without the learned correction)
  spmv      y = A x
  solve     BiCGSTAB to a relative residual of 1e-8
  setup     partition + ILU0 of a new matrix, and the first apply on it
  refactor  new values on a known pattern (time stepping), and an apply
  targets   the learned correction's regression targets: global ILU0 of the
            matrix and its apply on a batch of probes
  train     loss and gradient of one training problem

on three families of matrices: 7-point grid operators with 1x1 or 3x3 blocks
(Laplacians, random blocks, log-normal permeability fields, isotropic or
1:1:100) cut into boxes, and unstructured nearest-neighbour graphs cut by the
graph partitioner.  Every input is drawn on the GPU from the seed.
"""

from __future__ import annotations

import math

import numpy as np
import torch

from paper_2508_04917_amd import ddilu as dd
from paper_2508_04917_amd import lic

DEVICE = "cuda"
PRECISION = {"fp64": dd.DD_FP64, "mixed": dd.DD_MIXED, "fp32": dd.DD_FP32}
RTOL = 1e-8


def _case(name, op, kind, nx, ny, nz, bs=3, sub=0, precision="fp64", learned=False, nq=1, iters=0):
    """sub: edge of cubic boxes (0: the library's automatic choice); nq:
    probes of a training problem; iters: BiCGSTAB iterations such a solve
    takes (for the byte count alone)."""
    return {"name": name, "op": op, "kind": kind, "nx": nx, "ny": ny, "nz": nz, "bs": bs, "sub": sub,
            "precision": precision, "learned": learned, "nq": nq, "iters": iters}


def listed():
    return [
        # the smallest problem anyone solves: eight scalar boxes, all latency
        _case("solve_scalar_16", "solve", "laplacian", 16, 16, 16, bs=1, sub=8, iters=23),
        # one preconditioner apply inside someone else's Krylov method, a grid of moderate size
        _case("apply_blocks_64", "apply", "random", 64, 64, 64),
        # the same on the reservoir-sized grid the apply's bandwidth is quoted on
        _case("apply_lognormal_160", "apply", "lognormal", 160, 160, 160),
        # FP32 factors and the learned correction, on a ragged grid
        _case("apply_learned_ragged", "apply", "lognormal", 105, 132, 78, precision="mixed", learned=True),
        # a linear system of moderate size, plain FP64
        _case("solve_blocks_64", "solve", "random", 64, 64, 64, iters=177),
        # the headline configuration (learned correction, FP32 factors, FP64 Krylov) on an evaluation-sized grid
        _case("solve_learned_128", "solve", "lognormal", 128, 128, 128, precision="mixed", learned=True, iters=280),
        # a matrix without geometry, already partitioned: the whole solve
        _case("solve_graph_blocks", "solve", "graph", 160, 128, 100, iters=22),
        # a matrix without geometry, new: graph partition and factorisation
        _case("setup_graph_scalar", "setup", "graph", 128, 100, 80, bs=1),
        # a new matrix on a grid: partition and factorisation
        _case("setup_lognormal_128", "setup", "lognormal", 128, 128, 128),
        # the next time step: new values on the same grid, odd extents
        _case("refactor_aniso_ragged", "refactor", "aniso", 99, 80, 108),
        # training the learned correction: one problem's targets, then one of its gradient steps
        _case("targets_48", "targets", "lognormal", 48, 48, 48, sub=16, nq=16),
        _case("train_48", "train", "lognormal", 48, 48, 48, sub=16, nq=16),
    ]


def draw(rng):
    """One more case of the same ranges: any operation, any family it is used
    on, grid extents from 16 up to where the listed cases end."""
    def extent(lo, hi):
        # products of two moderate factors, so that boxes other than lines exist
        while True:
            e = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
            if lo <= e <= hi and any(e % f == 0 for f in range(4, 17) if e // f >= 2):
                return e

    op = rng.choice(["apply", "apply", "spmv", "solve", "setup", "refactor", "train", "targets"])
    if op in ("train", "targets"):
        s = rng.choice([6, 8, 12, 16])
        d = [s * rng.randint(2, max(2, 48 // s)) for _ in range(3)]
        return {k: v for k, v in _case("", op, "lognormal", *d, sub=s, nq=rng.randint(3, 16)).items() if k != "name"}
    kinds = ["laplacian", "random", "lognormal", "aniso", "graph"]
    if op == "solve":
        kinds = ["laplacian", "random", "graph"]
    if op == "refactor":
        kinds = ["random", "lognormal", "aniso"]
    kind = rng.choice(kinds)
    top = {"apply": 150, "spmv": 150, "solve": 80, "setup": 110, "refactor": 100}[op]
    d = [extent(16, top) for _ in range(3)]
    if kind == "graph":
        d = [8 * max(2, d[0] // 8), 4 * max(4, d[1] // 4), 4 * max(4, d[2] // 4)]
    bs = 3 if kind in ("random", "lognormal", "aniso") else rng.choice([1, 3])
    precision = rng.choice(["fp64", "mixed", "fp32"]) if op == "apply" else rng.choice(["fp64", "mixed"])
    if op in ("spmv", "setup", "refactor"):
        precision = "fp64"
    learned = kind in ("lognormal", "random") and op == "apply" and rng.random() < 0.4
    iters = {"laplacian": 60, "random": 100, "graph": 22}.get(kind, 0) if op == "solve" else 0
    c = _case("", op, kind, *d, bs=bs, precision=precision, learned=learned, iters=iters)
    return {k: v for k, v in c.items() if k != "name"}


# ------------------------------------------------------------------ inputs
def _grid(nx, ny, nz):
    """7-point pattern: neighbour of each cell in the seven directions
    (-z -y -x self +x +y +z), and which of them exist."""
    g = torch.arange(nx * ny * nz, device=DEVICE)
    i, j, k = g % nx, (g // nx) % ny, g // (nx * ny)
    off = torch.tensor([-nx * ny, -nx, -1, 0, 1, nx, nx * ny], device=DEVICE)
    ok = torch.stack([k > 0, j > 0, i > 0, torch.ones_like(i, dtype=torch.bool), i < nx - 1, j < ny - 1, k < nz - 1], 1)
    return g[:, None] + off, ok


def _randn(gen, *shape):
    return torch.randn(*shape, generator=gen, device=DEVICE, dtype=torch.float64)


def _eye(bs):
    return torch.eye(bs, device=DEVICE, dtype=torch.float64)


def _sym(gen, n, bs):
    G = _randn(gen, n, bs, bs)
    return 0.05 * (G + G.transpose(1, 2))


def _permeability(gen, nx, ny, nz, sigma=2.0, corr=8.0):
    """Log-normal field exp(sigma g), g Gaussian with correlation length corr cells."""
    w = _randn(gen, nz, ny, nx)
    s = corr / math.sqrt(2.0)
    f = [torch.fft.fftfreq(m, device=DEVICE, dtype=torch.float64) for m in (nz, ny, nx)]
    kern = torch.exp(-2.0 * math.pi ** 2 * s ** 2 * (f[0][:, None, None] ** 2 + f[1][:, None] ** 2 + f[2] ** 2))
    g = torch.fft.ifftn(torch.fft.fftn(w) * kern).real
    g = (g - g.mean()) / g.std()
    return torch.exp(sigma * g).reshape(-1)


def _grid_values(kind, nx, ny, nz, bs, nb, ok, gen):
    """Blocks [n, 7, bs, bs] of a grid operator (rows' missing neighbours hold zeros)."""
    n = nx * ny * nz
    if kind == "laplacian":
        v = (-_eye(bs)).repeat(n, 7, 1, 1)
        v[:, 3] = 6.0 * _eye(bs)
    elif kind == "random":
        v = 0.05 * _randn(gen, n, 7, bs, bs) - _eye(bs)
        v[:, 3] = 6.0 * _eye(bs) + _sym(gen, n, bs)
    else:  # two-point flux on a log-normal field: couplings -k_f (I - 0.05 H), rows summing to zero inside
        mult = torch.tensor([1.0, 1.0, 100.0 if kind == "aniso" else 1.0], device=DEVICE, dtype=torch.float64)
        axis = torch.tensor([2, 1, 0, 0, 0, 1, 2], device=DEVICE)
        k = _permeability(gen, nx, ny, nz)
        kb = k[nb.clamp(0, n - 1)]
        kf = mult[axis] * 2.0 * k[:, None] * kb / (k[:, None] + kb) * ok
        kf[:, 3] = 0.0
        v = _randn(gen, n, 7, bs, bs).mul_(0.05).sub_(_eye(bs)).mul_(kf[:, :, None, None])
        edge = (mult[axis] * ~ok).sum(1) * 2.0 * k
        v[:, 3] = -v.sum(1) + edge[:, None, None] * _eye(bs)
    return v


def _graph(nx, ny, nz, gen):
    """Nearest-neighbour graph of jittered points (six neighbours each,
    symmetrised, diagonal added) in a random numbering."""
    n = nx * ny * nz
    g = torch.arange(n, device=DEVICE)
    ijk = torch.stack([g % nx, (g // nx) % ny, g // (nx * ny)], 1)
    pt = ijk + torch.rand(n, 3, generator=gen, device=DEVICE)
    dist, cand = [], []
    for dz in (-1, 0, 1):
        for dy in (-1, 0, 1):
            for dx in (-1, 0, 1):
                if dx or dy or dz:
                    q = ijk + torch.tensor([dx, dy, dz], device=DEVICE)
                    ok = ((q >= 0) & (q < torch.tensor([nx, ny, nz], device=DEVICE))).all(1)
                    c = torch.where(ok, g + dx + nx * (dy + ny * dz), g)
                    d = (pt[c] - pt).square().sum(1)
                    dist.append(torch.where(ok, d, torch.full_like(d, 1e9)))
                    cand.append(c)
    near = torch.stack(dist, 1).topk(6, dim=1, largest=False).indices
    J = torch.stack(cand, 1).gather(1, near).reshape(-1)
    I = g.repeat_interleave(6)
    number = torch.randperm(n, generator=gen, device=DEVICE)
    I, J = number[I], number[J]
    keys = torch.unique(torch.cat([I * n + J, J * n + I, g * (n + 1)]))
    return keys // n, keys % n


def _matrix(case, seed, values=0):
    """Rows, columns and blocks of the case's matrix, on the GPU.  values: which
    draw of the values (the pattern does not depend on it)."""
    nx, ny, nz, bs, kind = (case[k] for k in ("nx", "ny", "nz", "bs", "kind"))
    gen = torch.Generator(device=DEVICE).manual_seed(10 * seed + 7 * values)
    if kind != "graph":
        nb, ok = _grid(nx, ny, nz)
        val = _grid_values(kind, nx, ny, nz, bs, nb, ok, gen)[ok]
        I = torch.arange(nb.shape[0], device=DEVICE).repeat_interleave(ok.sum(1))
        return I, nb[ok], val
    I, J = _graph(nx, ny, nz, gen)
    n = nx * ny * nz
    val = 0.05 * _randn(gen, I.numel(), bs, bs) - _eye(bs)
    d = I == J
    deg = torch.bincount(I, minlength=n) - 1
    val[d] = (deg + 0.5)[:, None, None] * _eye(bs) + _sym(gen, n, bs)
    return I, J, val


def _csr(I, J, val, n):
    ptr = torch.zeros(n + 1, dtype=torch.int32, device=DEVICE)
    ptr[1:] = torch.bincount(I, minlength=n).cumsum(0)
    return ptr, J.to(torch.int32), val.reshape(-1).contiguous()


def _vector(case, seed, count=1):
    """Right-hand sides or probes, N(0,1)."""
    gen = torch.Generator(device=DEVICE).manual_seed(10 * seed + 3)
    m = case["nx"] * case["ny"] * case["nz"] * case["bs"]
    v = _randn(gen, count, m)
    return v if count > 1 else v[0].contiguous()


def _params():
    return lic.load_params()[0]


# ---------------------------------------------------------- the user's program
def _partition(case, ptr, col, val):
    nx, ny, nz, bs, s = (case[k] for k in ("nx", "ny", "nz", "bs", "sub"))
    if case["kind"] == "graph":
        return dd.dd_partition_graph(nx * ny * nz, bs, ptr, col, val)
    return dd.dd_partition(nx, ny, nz, bs, ptr, col, val, sub=(s, s, s))


def prepare(case, seed):
    n = case["nx"] * case["ny"] * case["nz"]
    op = case["op"]
    ptr, col, val = _csr(*_matrix(case, seed), n)
    st = {"case": case, "op": op, "r": _vector(case, seed, case["nq"])}
    if op == "setup":
        st["matrix"] = (ptr, col, val)
        return st
    h = st["h"] = _partition(case, ptr, col, val)
    if op == "spmv":
        st["y"] = torch.empty_like(st["r"])
        return st
    dd.ilu0_factor(h, PRECISION[case["precision"]])
    if op in ("targets", "train") or case["learned"]:
        dd.lic_setup(h)
        st["params"] = torch.as_tensor(_params(), device=DEVICE)
    if case["learned"]:
        dd.lic_set_params(h, st["params"])
    if op == "refactor":
        st["values"] = _csr(*_matrix(case, seed, values=1), n)[2]
    if op == "train":
        dd.dd_global_factor(h)
        st["targets"], st["den"] = dd.lic_targets(h, st["r"])
    if op in ("apply", "refactor"):
        st["z"] = torch.empty_like(st["r"])
    return st


def run(st):
    op = st["op"]
    if op == "apply":
        return dd.dd_trsv_apply(st["h"], st["r"], st["z"])
    if op == "spmv":
        return dd.dd_spmv(st["h"], st["r"], st["y"])
    if op == "solve":
        x, info = dd.bicgstab_solve(st["h"], st["r"], rtol=RTOL, maxit=5000)
        return {"x": x, "iterations": info["iters"], "status": info["status"], "residual": info["rel_res"]}
    if op == "setup":
        h = _partition(st["case"], *st["matrix"])
        dd.ilu0_factor(h)
        z = dd.dd_trsv_apply(h, st["r"])
        h.close()
        return z
    if op == "refactor":
        dd.ilu0_refactor(st["h"], st["values"])
        return dd.dd_trsv_apply(st["h"], st["r"], st["z"])
    if op == "targets":
        dd.dd_global_factor(st["h"])
        Z, den = dd.lic_targets(st["h"], st["r"])
        return {"targets": Z, "den": den}
    loss, grad = dd.lic_loss_grad(st["h"], st["params"], st["r"], st["targets"], st["den"])
    return {"loss": loss, "grad": grad}


# --------------------------------------------------------------- work done
def work(case):
    nx, ny, nz, bs, op, nq = (case[k] for k in ("nx", "ny", "nz", "bs", "op", "nq"))
    n, bb = nx * ny * nz, bs * bs
    if case["kind"] == "graph":  # about 7.2 neighbours a row, one in ten of them cut
        off, kept = 7.2 * n, 6.5 * n
    else:
        off = 6.0 * n - 2.0 * (nx * ny + ny * nz + nz * nx)
        sx, sy, sz = _box(case)
        kept = 6.0 * n - 2.0 * n * (1.0 / sx + 1.0 / sy + 1.0 / sz)
    cut = off - kept
    w = 8 if case["precision"] == "fp64" else 4
    vec = 8.0 * n * bs
    matrix = (off + n) * (8.0 * bb + 4)
    factors = kept * (w * bb + 4.0) + n * bb * w
    apply_b = factors + 2 * vec + (cut * (4.0 * bb + 8) + 8.0 * bs * cut if case["learned"] else 0.0)
    apply_f = 2.0 * bb * (kept + n)
    spmv_b, spmv_f = matrix + 2 * vec, 2.0 * bb * (off + n)
    mlp = 2.0 * (27 * 64 + 64 * 64 + 64 * 9)
    if op == "apply":
        b, f = apply_b, apply_f
    elif op == "spmv":
        b, f = spmv_b, spmv_f
    elif op == "solve":  # per iteration two applies, two products, and the recurrence's vectors once each way
        b = case["iters"] * 2.0 * (apply_b + spmv_b + 5 * vec)
        f = case["iters"] * 2.0 * (apply_f + spmv_f + 6.0 * n * bs)
    elif op in ("setup", "refactor"):
        b, f = matrix + factors + apply_b, 4.0 * bs * bb * kept + apply_f
    elif op == "targets":
        b = matrix + 2 * (off * (8.0 * bb + 4) + n * bb * 8.0) + factors + 3 * nq * vec
        f = 4.0 * bs * bb * off + nq * 2.0 * (spmv_f + apply_f)
    else:  # forward and adjoint applies of every probe, MLP forward and backward on every cut face
        b = 2 * factors + 3 * nq * vec + cut * 4.0 * 27
        f = nq * 2.0 * apply_f + 3.0 * mlp * cut
    return {"bytes": b, "flops": f}


# ------------------------------------------------- plain 64-bit evaluation
def _box(case):
    """Box extents: the given edge, or the largest box of grid divisors whose
    vector fits 160 KB with at least one box per compute unit (then the
    smallest surface, largest sz, sy)."""
    nx, ny, nz, bs, s = (case[k] for k in ("nx", "ny", "nz", "bs", "sub"))
    if s:
        return s, s, s
    div = lambda m: [d for d in range(1, m + 1) if m % d == 0]  # noqa: E731
    fit = [(x, y, z) for x in div(nx) for y in div(ny) for z in div(nz) if x * y * z * bs * 8 <= 163840]
    full = [b for b in fit if nx * ny * nz // (b[0] * b[1] * b[2]) >= 256]
    return max(full or fit, key=lambda b: (b[0] * b[1] * b[2], -(b[0] * b[1] + b[1] * b[2] + b[2] * b[0]), b[2], b[1]))


def _mul(A, B):
    return (A[:, :, :, None] * B[:, None, :, :]).sum(2)


def _inverse(a):
    if a.shape[-1] == 1:
        return 1.0 / a
    c = torch.stack([torch.linalg.cross(a[:, 1], a[:, 2]), torch.linalg.cross(a[:, 2], a[:, 0]),
                     torch.linalg.cross(a[:, 0], a[:, 1])], 2)
    return c / (a[:, 0] * c[:, :, 0]).sum(1)[:, None, None]


class _Ilu0:
    """ILU0 of a pattern without triangles (a 7-point operator in any
    numbering: only the diagonal blocks change), rows level by level."""

    def __init__(self, I, J, A, n):
        self.n = n
        d = I == J
        keys = I * n + J
        rev = torch.searchsorted(keys, J * n + I)
        self.parts = []
        for e in (J < I, J > I):
            e = e.nonzero()[:, 0]
            lev = torch.zeros(n, dtype=torch.int64, device=DEVICE)
            while True:
                new = torch.zeros_like(lev).scatter_reduce_(0, I[e], lev[J[e]] + 1, "amax")
                if torch.equal(new, lev):
                    break
                lev = new
            o = torch.argsort(lev[I[e]], stable=True)
            rows = torch.argsort(lev, stable=True)
            top = int(lev.max()) + 1
            self.parts.append((e[o], torch.bincount(lev[I[e]], minlength=top).cumsum(0).tolist(), rows,
                               torch.bincount(lev, minlength=top).cumsum(0).tolist()))
        self.I, self.J, self.A, self.rev = I, J, A, rev
        D = torch.empty(n, *A.shape[1:], dtype=torch.float64, device=DEVICE)
        D[I[d]] = A[d]
        self.inv = torch.empty_like(D)
        for e, rows in self._levels(0):
            if e.numel():
                D.index_add_(0, I[e], _mul(_mul(A[e], self.inv[J[e]]), A[rev[e]]), alpha=-1.0)
            self.inv[rows] = _inverse(D[rows])

    def _levels(self, which):
        e, eo, rows, ro = self.parts[which]
        for l in range(len(ro)):
            yield e[eo[l - 1] if l else 0:eo[l]], rows[ro[l - 1] if l else 0:ro[l]]

    def solve(self, r):
        """r [n, bs, q] -> M^{-1} r."""
        y, inv = r.clone(), self.inv
        for e, _ in self._levels(0):
            if e.numel():
                y.index_add_(0, self.I[e], _mul(self.A[e], _mul(inv[self.J[e]], y[self.J[e]])), alpha=-1.0)
            # y holds L^{-1} r: L_IJ = A_IJ inv(U_JJ)
        for e, rows in self._levels(1):
            if e.numel():
                y.index_add_(0, self.I[e], _mul(self.A[e], y[self.J[e]]), alpha=-1.0)
            y[rows] = _mul(inv[rows], y[rows])
        return y

    def solve_transposed(self, g):
        w, inv, t = g.clone(), self.inv, lambda a: a.transpose(1, 2)
        for e, rows in self._levels(0):
            if e.numel():
                w.index_add_(0, self.I[e], _mul(t(self.A[self.rev[e]]), w[self.J[e]]), alpha=-1.0)
            w[rows] = _mul(t(inv[rows]), w[rows])
        for e, _ in self._levels(1):
            if e.numel():
                w.index_add_(0, self.I[e], _mul(t(inv[self.I[e]]), _mul(t(self.A[self.rev[e]]), w[self.J[e]])),
                             alpha=-1.0)
        return w


def _reordered(case, seed, values=0):
    """The matrix in the library's numbering (boxes one after another, cells of
    a box in lexicographic order), sorted by row and column; box of each row."""
    nx, ny, nz = (case[k] for k in ("nx", "ny", "nz"))
    sx, sy, sz = _box(case)
    I, J, A = _matrix(case, seed, values)
    g = torch.arange(nx * ny * nz, device=DEVICE)
    i, j, k = g % nx, (g // nx) % ny, g // (nx * ny)
    box = i // sx + (nx // sx) * (j // sy + (ny // sy) * (k // sz))
    new = box * (sx * sy * sz) + i % sx + sx * (j % sy + sy * (k % sz))
    I, J = new[I], new[J]
    o = torch.argsort(I * g.numel() + J)
    I, J = I[o], J[o]
    S = sx * sy * sz
    return I, J, A[o], I // S == J // S


def _correction(I, J, A, inside, P):
    """Faces and their coefficients: the MLP on the blocks at each cut."""
    f = (~inside).nonzero()[:, 0]
    D = A[I == J]
    Aii, Ajj = D[I[f]], D[J[f]]
    tr = lambda b: b.diagonal(dim1=1, dim2=2).sum(1).abs()  # noqa: E731
    s = torch.sqrt(tr(Aii) * tr(Ajj)) / 3.0
    x = torch.cat([b.reshape(-1, 9) / s[:, None] for b in (Aii, A[f], Ajj)], 1)
    w, at = [], 0
    for rows, cols in ((64, 27), (64, 64), (9, 64)):
        w.append((P[at:at + rows * cols].view(rows, cols), P[at + rows * cols:at + rows * cols + rows]))
        at += rows * cols + rows
    for k, (W, b) in enumerate(w):
        x = x @ W.T + b
        x = torch.relu(x) if k < 2 else x
    return f, x.view(-1, 3, 3)


def _exact_apply(case, seed, r, values=0):
    I, J, A, inside = _reordered(case, seed, values)
    if case["learned"]:
        P = torch.as_tensor(_params(), device=DEVICE).double()
        f, C = _correction(I, J, A, inside, P)
        r = r.index_add(0, I[f], _mul(C, r[J[f]]))
    return _Ilu0(I[inside], J[inside], A[inside], r.shape[0]).solve(r)


def _exact_solution(I, J, A, b):
    """BiCGSTAB with block-diagonal scaling to a residual at rounding level, or None."""
    n, bs = b.numel() // A.shape[-1], A.shape[-1]
    inv = _inverse(A[I == J])

    def mul(x):
        x = _mul(inv, x.view(n, bs, 1))
        y = torch.zeros(n, bs, 1, dtype=torch.float64, device=DEVICE)
        return y.index_add_(0, I, _mul(A, x[J])).reshape(-1)

    total = torch.zeros_like(b)
    r = b.clone()
    for _ in range(4):  # restarts bring the true residual down
        x, r0, p = torch.zeros_like(b), r.clone(), r.clone()
        rho = r0 @ r
        for _ in range(400):
            v = mul(p)
            a = rho / (r0 @ v)
            s = r - a * v
            t = mul(s)
            om = (t @ s) / (t @ t)
            x += a * p + om * s
            r = s - om * t
            if float(r.norm() / b.norm()) < 1e-13:
                break
            new = r0 @ r
            p = r + (new / rho) * (a / om) * (p - om * v)
            rho = new
        if not bool(torch.isfinite(x).all()):
            return None
        total += x
        r = b - mul(total)
        if float(r.norm() / b.norm()) < 2e-13:
            return _mul(inv, total.view(n, bs, 1)).reshape(-1)
    return None


def exact(case, seed):
    op, bs, kind, n = case["op"], case["bs"], case["kind"], case["nx"] * case["ny"] * case["nz"]
    r = _vector(case, seed, case["nq"])
    if op == "solve":
        # the field problems need the preconditioner to converge at all
        x = None if kind in ("lognormal", "aniso") else _exact_solution(*_matrix(case, seed), r)
        return None if x is None else {"x": x, "iterations": None, "status": None, "residual": None}
    if kind == "graph":
        return None  # the numbering is the partitioner's own
    R = r.view(-1, n, bs).permute(1, 2, 0).contiguous()
    flat = lambda z: z.permute(2, 0, 1).reshape(r.shape)  # noqa: E731
    if op in ("apply", "setup"):
        return flat(_exact_apply(case, seed, R))
    if op == "refactor":
        return flat(_exact_apply(case, seed, R, values=1))
    I, J, A, inside = _reordered(case, seed)
    if op == "spmv":
        return flat(torch.zeros_like(R).index_add_(0, I, _mul(A, R[J])))
    Z = _Ilu0(I, J, A, n).solve(R)
    M = _Ilu0(I[inside], J[inside], A[inside], n)
    den = (M.solve(R) - Z).square().sum((0, 1))
    if op == "targets":
        return {"targets": flat(Z), "den": den}
    P = torch.as_tensor(_params(), device=DEVICE).double().requires_grad_(True)
    f, C = _correction(I, J, A, inside, P)
    E = M.solve(R.index_add(0, I[f], _mul(C.detach(), R[J[f]]))) - Z
    nq = case["nq"]
    loss = (E.square().sum((0, 1)) / den).sum() / nq
    a = M.solve_transposed(2.0 * E / (nq * den))
    dC = (a[I[f]][:, :, None, :] * R[J[f]][:, None, :, :]).sum(3)
    C.backward(dC)
    return {"loss": loss.reshape(1), "grad": np.asarray(P.grad.cpu())}
