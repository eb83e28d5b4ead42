"""The work that users of this library have it do, as cases that can be timed and checked.

A case names a scene (a seeded synthetic mesh with its terms), its size, a precision and what is asked of the
library: the energy with gradient and (clamped) Hessian, a matrix-free product, a sparse Jacobian, or a training
step of the learned density. ``exact`` states the same energies once more in plain FP64 torch (hyper-dual
arithmetic over whole batches of elements, a Jacobi eigen-solver, a sorted union for the block pattern).
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

from paper_2509_00406_amd import mad

E, G, H, SPD = mad.ENERGY, mad.GRAD, mad.HESS, mad.SPD
KB, MU, LAM, CLOTH_K, CLOTH_H = 1.0, 1.0, 1.0, 1.0e3, 1.0 / 60.0
GRAVITY = (0.0, 0.0, -9.81)


def listed():
    return [
        # the smallest call: a scalar Dirichlet energy on 64 x 64 vertices, where launches are all there is
        dict(name="dirichlet_64_f64", scene="dirichlet", n=64, prec="f64", ask="hess"),
        # a Newton step of a small elastic shell, the size of an interactive simulation (odd side)
        dict(name="shell_101_f32", scene="shell", n=101, prec="f32", ask="spd"),
        # the benchmark: membrane and bending of a 1024 x 1024 shell, filtered for Newton's method
        dict(name="shell_1024_f32", scene="shell", n=1024, prec="f32", ask="spd"),
        # the same energies in double precision on a million triangles
        dict(name="shell_708_f64", scene="shell", n=708, prec="f64", ask="spd"),
        # an implicit-Euler step of a mass-spring cloth: cheap elements, memory and latency
        dict(name="cloth_1000_f32", scene="cloth", n=1000, prec="f32", ask="spd"),
        # area smoothing by gradient descent: energy and gradient only
        dict(name="area_grad_500_f32", scene="area", n=500, prec="f32", ask="grad"),
        # projected Newton for a parameterisation with two unknowns per vertex
        dict(name="symdir_1001_f32", scene="symdir", n=1001, prec="f32", ask="spd"),
        # one conjugate-gradient product of the same energy without assembling its Hessian
        dict(name="symdir_hvp_748_f32", scene="symdir", n=748, prec="f32", ask="hvp"),
        # many bodies in one launch: disjoint shells of different sizes, an energy for each
        dict(name="spheres_700_f32", scene="spheres", n=700, prec="f32", ask="spd"),
        # the learned per-triangle density (stored network) on a million triangles
        dict(name="learned_708_f32", scene="learned", n=708, prec="f32", ask="spd"),
        # residuals and sparse Jacobian of a Gauss-Newton solve
        dict(name="jacobian_1000_f32", scene="residual", n=1000, prec="f32", ask="jacobian"),
        # one optimiser step of the learned density at the training recipe's minibatch
        dict(name="train_512", scene="train", n=512, prec="f32", ask="train"),
    ]


def draw(rng):
    def size(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    scene = rng.choice(["shell", "shell", "cloth", "symdir", "symdir", "spheres", "learned", "residual", "train",
                        "dirichlet", "area"])
    prec = rng.choice(["f32", "f32", "f64"])
    if scene == "train":
        return dict(scene=scene, n=size(32, 2048), prec="f32", ask="train")
    if scene == "residual":
        return dict(scene=scene, n=size(16, 1000), prec=prec, ask="jacobian")
    if scene == "spheres":
        return dict(scene=scene, n=size(1, 700 if prec == "f32" else 200), prec=prec, ask="spd")
    top = dict(shell=1024, cloth=1000, symdir=1001, learned=708, dirichlet=1000, area=1000)[scene]
    if prec == "f64" and scene == "shell":
        top = 500
    low = dict(shell=10, cloth=10, symdir=39, learned=16, dirichlet=16, area=16)[scene]
    ask = rng.choice(dict(shell=["spd", "spd", "hess", "grad", "hvp"], cloth=["spd"], symdir=["spd", "hvp"],
                          learned=["spd"], dirichlet=["hess"], area=["grad"])[scene])
    return dict(scene=scene, n=size(low, top), prec=prec, ask=ask)


# ---- inputs (from the seed alone) ---------------------------------------------------------------
@functools.lru_cache(maxsize=16)
def _grid(n):
    """n x n vertices on the unit square, each square cut along the same diagonal: triangles, positions."""
    t = np.arange(n) / (n - 1)
    pos = np.zeros((n * n, 3))
    pos[:, 0], pos[:, 1] = np.tile(t, n), np.repeat(t, n)
    v = (np.arange(n - 1)[:, None] * n + np.arange(n - 1)[None, :]).ravel()
    tris = np.stack([v, v + 1, v + n + 1, v, v + n + 1, v + n], axis=1).reshape(-1, 3).astype(np.int32)
    return tris, pos


@functools.lru_cache(maxsize=64)
def _icosphere(f):
    """Unit geodesic sphere of frequency f: 20 f^2 triangles facing outward, 10 f^2 + 2 vertices."""
    g = (1 + math.sqrt(5)) / 2
    c = np.array([[0, s, t * g] for s in (-1, 1) for t in (-1, 1)], float)
    c = np.concatenate([c, c[:, [2, 0, 1]], c[:, [1, 2, 0]]]) / math.sqrt(1 + g * g)
    near = (c @ c.T) > 0.4
    faces = [(i, j, k) for i in range(12) for j in range(i + 1, 12) for k in range(j + 1, 12)
             if near[i, j] and near[j, k] and near[i, k]]
    ij = [(i, j) for j in range(f + 1) for i in range(f + 1 - j)]
    at = {p: k for k, p in enumerate(ij)}
    up = [(at[i, j], at[i + 1, j], at[i, j + 1]) for i, j in ij if i + j < f]
    down = [(at[i + 1, j], at[i + 1, j + 1], at[i, j + 1]) for i, j in ij if i + j < f - 1]
    w = np.array([(f - i - j, i, j) for i, j in ij]) / f
    pts = np.concatenate([w @ c[list(t)] for t in faces])
    tri = np.array(up + down)
    tris = np.concatenate([tri + k * len(ij) for k in range(20)])
    _, first, inverse = np.unique(np.round(pts * 1e7).astype(np.int64), axis=0, return_index=True, return_inverse=True)
    pos = pts[first]
    pos /= np.linalg.norm(pos, axis=1, keepdims=True)
    tris = inverse.reshape(-1)[tris].astype(np.int32)
    a, b, d = pos[tris[:, 0]], pos[tris[:, 1]], pos[tris[:, 2]]
    flip = np.einsum("ij,ij->i", np.cross(b - a, d - a), a) < 0
    tris[flip] = tris[flip][:, [0, 2, 1]]
    return tris, pos


def _waves(p, rng, amplitude, dim, low, high, count):
    out = np.zeros((p.shape[0], dim))
    for _ in range(count):
        a = rng.normal(size=dim)
        g, r, phi = rng.uniform(0, 2 * math.pi), rng.uniform(low, high), rng.uniform(0, 2 * math.pi)
        s = np.sin(2 * math.pi * r * (p @ np.array([math.cos(g), math.sin(g)])) + phi)
        out += np.outer(s, a * (amplitude / count / np.linalg.norm(a)))
    return out


def _inputs(case, seed):
    """Mesh, rest positions, unknowns and further per-vertex data of a scene, as numpy arrays."""
    rng = np.random.default_rng([seed, case["n"]])
    scene, n = case["scene"], case["n"]
    d = dict(comp=None)
    if scene == "spheres":
        # geodesic spheres of lognormal size (mean 3,000 vertices), squashed, with small noise
        # (the sizes are the scene's own, the shapes the seed's)
        sizes = np.exp(np.random.default_rng(4001).normal(math.log(3000.0) - 0.125, 0.5, n)).clip(500, 12000)
        tris, rest, x, comp = [], [], [], [0]
        for m in range(n):
            t, p = _icosphere(min(34, max(8, round(math.sqrt((sizes[m] - 2) / 10)))))
            p = p * rng.uniform(0.5, 1.5)
            c = np.array([3.5 * (m % 27), 3.5 * (m // 27), 0.0])
            edge = np.linalg.norm(p[t[0, 0]] - p[t[0, 1]])
            tris.append(t + comp[-1])
            rest.append(p + c)
            x.append(p * (1.1, 1.1, 0.8) + rng.normal(0, 1e-3 * edge, p.shape) + c)
            comp.append(comp[-1] + p.shape[0])
        d.update(tris=np.concatenate(tris), rest=np.concatenate(rest), x=np.concatenate(x), comp=np.array(comp))
        return d
    tris, rest = _grid(n)
    h = 1.0 / (n - 1)
    if scene in ("shell", "learned"):   # a flat sheet rolled into a half cylinder, with small noise
        r = 1 / math.pi
        x = np.stack([r * np.sin(rest[:, 0] / r), rest[:, 1], r * (1 - np.cos(rest[:, 0] / r))], axis=1)
        x += rng.normal(0, 1e-3 * h, x.shape)
    elif scene == "dirichlet":          # jittered planar mesh, a random scalar per vertex
        rest = rest.copy()
        rest[:, :2] += rng.uniform(-0.2 * h, 0.2 * h, (n * n, 2))
        x = rng.standard_normal((n * n, 1))
    elif scene == "symdir":             # a smooth warp of the square that flips no triangle
        x = rest[:, :2] + _waves(rest[:, :2], rng, 0.1, 2, 0.5, 1.0, 8)
    elif scene == "area":               # a bumpy sheet
        x = rest + _waves(rest[:, :2], rng, 0.1, 3, 0.5, 2.0, 6) + rng.normal(0, 0.1 * h, rest.shape)
    elif scene == "cloth":              # stretched and compressed springs, smooth velocities
        x = rest + _waves(rest[:, :2], rng, 0.02, 3, 0.5, 2.0, 6)
        v = _waves(rest[:, :2], rng, 0.5, 3, 0.5, 2.0, 6)
        d["vdata"] = np.concatenate([np.full((n * n, 1), 1.0 / (n * n)), x + CLOTH_H * v], axis=1)
    elif scene == "residual":           # a quarter of the vertices pulled toward targets
        x = rest + rng.normal(0, 0.2 * h, rest.shape)
        w = np.where(rng.uniform(size=n * n) < 0.25, rng.uniform(0.5, 2.0, n * n), 0.0)
        d["vdata"] = np.concatenate([w[:, None], rest + (0, 0, 0.2) + rng.normal(0, 0.05, rest.shape)], axis=1)
    if case["ask"] == "hvp":
        d["v"] = rng.standard_normal(x.shape)
    d.update(tris=tris, rest=rest, x=x)
    return d


def _train_inputs(case, seed):
    """Samples (features, density, its gradient), scales and initial weights of a training run."""
    rng = np.random.default_rng([seed, case["n"]])
    z = rng.normal(size=(16 * case["n"], 6)) * (1e-2, 1e-2, 1e-2, 0.3, 0.3, 0.3)
    tr = z[:, 0] + z[:, 1]
    W = z[:, 0]**2 + z[:, 1]**2 + 2 * z[:, 2]**2 + 0.5 * tr**2 + 0.5 * (z[:, 3]**2 + z[:, 4]**2 + 2 * z[:, 5]**2)
    dW = z * (2, 2, 4, 1, 1, 2)
    dW[:, :2] += tr[:, None]
    z, W, dW = (a.astype(np.float32) for a in (z, W, dW))
    curv = np.array([3.0, 3.0, 4.0, 1.0, 1.0, 2.0])
    s_in = np.sqrt(curv / np.max(curv * z.var(axis=0))).astype(np.float32)
    theta = np.concatenate([rng.normal(0, 0.5, 384), rng.normal(0, 0.5, 64), rng.normal(0, 0.125, 4096),
                            rng.normal(0, 0.5, 64), rng.normal(0, 0.0625, 64), [0.0]]).astype(np.float32)
    return dict(z=z, W=W, dW=dW, s_in=s_in, s_out=float(np.float32(W.std())), c_e=float(np.float32(W.var())),
                c_g=(dW.astype(float)**2).mean(axis=0).astype(np.float32), theta=theta,
                perm=rng.permutation(z.shape[0]).astype(np.int32))


# ---- one pass through the library ----------------------------------------------------------------
MODES = dict(hess=E | G | H, spd=E | G | H | SPD, grad=E | G, hvp=SPD)


def prepare(case, seed):
    if case["ask"] == "train":
        d = _train_inputs(case, seed)
        net = mad.Network(d["theta"], d["s_in"], d["s_out"])
        dev = {k: torch.from_numpy(d[k]).cuda() for k in ("z", "W", "dW", "perm")}
        return dict(ask="train", net=net, batch=case["n"], at=0, c_e=d["c_e"], c_g=d["c_g"], **dev)
    d = _inputs(case, seed)
    mesh = mad.Mesh(d["tris"], d["rest"].shape[0], d["comp"])
    prob = mad.Problem(mesh, d["x"].shape[1], mad.F32 if case["prec"] == "f32" else mad.F64)
    scene = case["scene"]
    if scene in ("shell", "spheres"):
        prob.add_term(mad.STVK, (MU, LAM), d["rest"])
        prob.add_term(mad.BENDING, (KB, 1.0), d["rest"])
    elif scene == "learned":
        prob.add_mlp_term(mad.Network.from_file(), d["rest"])
    elif scene == "cloth":
        prob.add_term(mad.SPRING, (CLOTH_K, CLOTH_H**2), d["rest"])
        prob.add_vertex_term(mad.INERTIA, (CLOTH_H**2, *GRAVITY), torch.from_numpy(d["vdata"]).cuda())
    elif scene == "residual":
        prob.add_term(mad.RES_EDGE, (3.0,), d["rest"])
        prob.add_vertex_term(mad.RES_POSITION, (), torch.from_numpy(d["vdata"]).cuda())
    else:
        kind = dict(dirichlet=mad.DIRICHLET, symdir=mad.SYMDIR, area=mad.TRI_AREA)[scene]
        prob.add_term(kind, (), None if scene == "area" else d["rest"])
    prob.finalize()
    state = dict(ask=case["ask"], prob=prob, x=torch.from_numpy(d["x"]).cuda())
    if case["ask"] == "hvp":
        state["v"] = torch.from_numpy(d["v"]).cuda()
    if case["ask"] != "jacobian":
        state["out"] = prob.outputs()
    return state


def run(state):
    ask = state["ask"]
    if ask == "train":
        net, b = state["net"], state["batch"]
        grad, loss = net.loss_grad(state["z"], state["W"], state["dW"], state["c_e"], state["c_g"], 1.0,
                                   idx=state["perm"], base=state["at"], count=b)
        net.adam_step(grad, 1e-4)
        state["at"] = (state["at"] + b) % state["perm"].shape[0]
        return grad, loss
    prob = state["prob"]
    if ask == "jacobian":
        return prob.jacobian(state["x"])
    if ask == "hvp":
        return prob.hvp(state["x"], state["v"], SPD, state["out"])[0]
    out = prob.eval(state["x"], MODES[ask], state["out"])
    return out[:2] if ask == "grad" else out


def _counts(case):
    """vertices, triangles, edges, interior edges"""
    n = case["n"]
    if case["scene"] == "spheres":
        return 2990 * n, 5976 * n, 8964 * n, 8964 * n
    return n * n, 2 * (n - 1)**2, (n - 1) * (3 * n - 1), (n - 1) * (3 * n - 1) - 4 * (n - 1)


def work(case):
    """Unknowns, connectivity and rest data read once, outputs written once; for the arithmetic, some 30 k^2 for
    the derivatives of an element with k coordinates and 9 k^3 for its eigen-decomposition."""
    if case["ask"] == "train":
        b = case["n"]
        return dict(bytes=b * 52 + 4673 * 4 * 8, flops=b * 3 * 7 * 2 * (64 * 64 + 64 * 7))
    nv, nt, ne, ni = _counts(case)
    scene, ask, s = case["scene"], case["ask"], 4 if case["prec"] == "f32" else 8
    if ask == "jacobian":
        return dict(bytes=nv * (24 + 32 + 24 + 9 * s) + ne * (8 + 8 + 8 + 6 * s), flops=ne * 60 + nv * 30)
    d = dict(dirichlet=1, symdir=2).get(scene, 3)
    blocks = nv + 2 * ne + (2 * ni if scene in ("shell", "spheres") else 0)
    read = nv * d * 8 + dict(cloth=ne * 24 + nv * 32, area=nt * 12, learned=nt * 76).get(scene, nt * 52)
    wrote = dict(grad=nv * d * s, hvp=nv * d * (s + 8)).get(ask, nv * d * s + blocks * d * d * s)
    elems = dict(dirichlet=[(nt, 2)], symdir=[(nt, 4)], cloth=[(ne, 3), (nv, 3)]).get(scene, [(nt, 6)])
    if scene in ("shell", "spheres"):
        read += ni * 32
        elems.append((ni, 9))
    f = sum(c * (30 * k * (1 if ask == "grad" else k) + (9 * k**3 if ask in ("spd", "hvp") else 0)) for c, k in elems)
    return dict(bytes=read + wrote, flops=f + (nt * 68224 if scene == "learned" else 0))


# ---- the same in plain FP64 ----------------------------------------------------------------------
class _HD:
    """value [N], gradient [K, N] and Hessian [K, K, N] of a batch of elements"""

    def __init__(self, v, g, h):
        self.v, self.g, self.h = v, g, h

    def __add__(self, o):
        return _HD(self.v + o.v, self.g + o.g, self.h + o.h) if isinstance(o, _HD) else _HD(self.v + o, self.g, self.h)

    def __sub__(self, o):
        return self + o * -1.0 if isinstance(o, _HD) else self + (-o)

    def __mul__(self, o):
        if not isinstance(o, _HD):
            return _HD(self.v * o, self.g * o, self.h * o)
        c = self.g[:, None] * o.g[None]
        return _HD(self.v * o.v, self.v * o.g + o.v * self.g, self.v * o.h + o.v * self.h + c + c.transpose(0, 1))

    def chain(self, f, f1, f2):
        return _HD(f, f1 * self.g, f1 * self.h + f2 * (self.g[:, None] * self.g[None]))

    def sqrt(self):
        s = self.v.sqrt()
        return self.chain(s, 0.5 / s, -0.25 / (s * self.v))

    def recip(self):
        r = 1.0 / self.v
        return self.chain(r, -r * r, 2 * r**3)


def _angle(y, x):
    """atan2 of two batches"""
    r2 = y.v**2 + x.v**2
    py, px, pxy, pyy = x.v / r2, -y.v / r2, (y.v**2 - x.v**2) / r2**2, -2 * x.v * y.v / r2**2
    c = y.g[:, None] * x.g[None]
    d = y.g[:, None] * y.g[None] - x.g[:, None] * x.g[None]
    h = py * y.h + px * x.h + pyy * d + pxy * (c + c.transpose(0, 1))
    return _HD(torch.atan2(y.v, x.v), py * y.g + px * x.g, h)


def _dot(a, b):
    s = a[0] * b[0]
    for p, q in zip(a[1:], b[1:]):
        s = s + p * q
    return s


def _cross(a, b):
    return [a[1] * b[2] - a[2] * b[1], a[2] * b[0] - a[0] * b[2], a[0] * b[1] - a[1] * b[0]]


def _clamp(A):
    """max(lambda, 0) of symmetric [K, K, N] batches, by cyclic Jacobi rotations"""
    K = A.shape[0]
    V = torch.eye(K, dtype=A.dtype, device=A.device)[:, :, None].repeat(1, 1, A.shape[2])
    A = A.clone()
    norm = A.square().sum((0, 1))
    for _ in range(30):
        off = sum(A[p, q].square() for p in range(K) for q in range(p))
        if K == 1 or bool((off <= 1e-31 * norm).all()):
            break
        for p in range(K):
            for q in range(p + 1, K):
                a, d = A[p, q], A[q, q] - A[p, p]
                den = d.abs() + torch.sqrt(d * d + 4 * a * a)
                t = torch.where(den > 0, 2 * a / torch.where(den > 0, den, 1.0), 0.0) * torch.where(d < 0, -1.0, 1.0)
                c = 1 / torch.sqrt(1 + t * t)
                s = t * c
                for M in (A, V):
                    u, w = M[p].clone(), M[q]
                    M[p] = c * u - s * w
                    M[q] = s * u + c * w
                u, w = A[:, p].clone(), A[:, q]
                A[:, p] = c * u - s * w
                A[:, q] = s * u + c * w
    lam = torch.diagonal(A).t().clamp(min=0)
    out = torch.zeros_like(A)
    for m in range(K):   # rows of V are the eigenvectors
        out += (lam[m] * V[m])[:, None] * V[m][None]
    return out


def _frames(tris, rest):
    """inverse rest matrix (m00, m01, m11; lower entry 0) and area of every triangle"""
    a, b, c = (rest[tris[:, k]] for k in range(3))
    e1, e2 = b - a, c - a
    l1 = e1.norm(dim=1)
    x2 = (e1 * e2).sum(1) / l1
    area2 = torch.linalg.cross(e1, e2).norm(dim=1)
    y2 = area2 / l1
    return 1 / l1, -x2 / (l1 * y2), 1 / y2, 0.5 * area2


def _edges(tris, nv):
    """edges (i < j) in ascending order; diamonds of the edges with two faces and those faces"""
    t = tris.long()
    i, j, k = (torch.cat([t[:, s % 3] for s in r]) for r in ((0, 1, 2), (1, 2, 3), (2, 3, 4)))
    face = torch.arange(t.shape[0], device=t.device).repeat(3)
    key = torch.minimum(i, j) * nv + torch.maximum(i, j)
    key, order = torch.sort(key, stable=True)
    i, j, k, face = i[order], j[order], k[order], face[order]
    first = torch.ones_like(key, dtype=torch.bool)
    first[1:] = key[1:] != key[:-1]
    start = torch.nonzero(first).ravel()
    count = torch.diff(torch.cat([start, torch.tensor([key.numel()], device=key.device)]))
    s = start[count == 2]
    lo = torch.where(face[s] < face[s + 1], s, s + 1)
    hi = 2 * s + 1 - lo
    return (torch.stack([key[start] // nv, key[start] % nv], 1), torch.stack([i[lo], j[lo], k[lo], k[hi]], 1), face[s],
            face[s + 1])


def _dihedral(p, q):
    """signed angle of diamonds given by four lists of three coordinates each; q: HD or plain arithmetic"""
    e, a, b = ([q(u, w) for u, w in zip(p[s], p[0])] for s in (1, 2, 3))
    n1, n2 = _cross(e, a), _cross(b, e)
    return e, n1, n2, b


def _terms(case, d):
    """[(stencils [N, NS], element energy of a list of NS * D unknowns and the elements' numbers)]"""
    tris, rest = d["tris"].long(), d["rest"]
    nv, scene = rest.shape[0], case["scene"]
    edges, dia, f0, f1 = _edges(tris, nv)
    m00, m01, m11, area = _frames(tris, rest)

    def strain(x, k):
        r1, r2 = [x[3 + c] - x[c] for c in range(3)], [x[6 + c] - x[c] for c in range(3)]
        a = [r * m00[k] for r in r1]
        b = [p * m01[k] + q * m11[k] for p, q in zip(r1, r2)]
        return a, b, (_dot(a, a) + -1.0) * 0.5, (_dot(b, b) + -1.0) * 0.5, _dot(a, b) * 0.5

    def stvk(x, k):
        _, _, e0, e1, e2 = strain(x, k)
        tr = e0 + e1
        return ((e0 * e0 + e1 * e1 + e2 * e2 * 2.0) * MU + tr * tr * (0.5 * LAM)) * area[k]

    def bend(x, k):
        e, n1, n2, b = _dihedral([x[3 * s:3 * s + 3] for s in range(4)], lambda u, w: u - w)
        t = _angle(_dot(e, e).sqrt() * _dot(n1, b) * -1.0, _dot(n1, n2)) - rest_angle[k]
        return t * t * (KB / 6.0 * (area[f0[k]] + area[f1[k]]))

    if scene in ("shell", "spheres"):
        p = [[rest[dia[:, s], c] for c in range(3)] for s in range(4)]
        e, n1, n2, b = _dihedral(p, lambda u, w: u - w)
        rest_angle = torch.atan2(-_dot(e, e).sqrt() * _dot(n1, b), _dot(n1, n2))
        return [(tris, stvk), (dia, bend)]
    if scene == "dirichlet":
        def energy(x, k):
            g0 = (x[1] - x[0]) * m00[k]
            g1 = (x[1] - x[0]) * m01[k] + (x[2] - x[0]) * m11[k]
            return (g0 * g0 + g1 * g1) * (0.5 * area[k])
        return [(tris, energy)]
    if scene == "symdir":
        def energy(x, k):
            r1, r2 = [x[2 + c] - x[c] for c in range(2)], [x[4 + c] - x[c] for c in range(2)]
            a, b = [r * m00[k] for r in r1], [p * m01[k] + q * m11[k] for p, q in zip(r1, r2)]
            det, n = a[0] * b[1] - a[1] * b[0], _dot(a, a) + _dot(b, b)
            return (n + n * (det * det).recip()) * area[k]
        return [(tris, energy)]
    if scene == "area":
        def energy(x, k):
            n = _cross([x[3 + c] - x[c] for c in range(3)], [x[6 + c] - x[c] for c in range(3)])
            return _dot(n, n).sqrt() * 0.5
        return [(tris, energy)]
    if scene == "cloth":
        l2 = (rest[edges[:, 0]] - rest[edges[:, 1]]).square().sum(1)

        def spring(x, k):
            r = [x[3 + c] - x[c] for c in range(3)]
            q = _dot(r, r) * (1 / l2[k]) + -1.0
            return q * q * (0.5 * CLOTH_K * CLOTH_H**2 * l2[k])

        def inertia(x, k):
            m, xh = d["vdata"][k, 0], d["vdata"][k, 1:]
            r = [x[c] - xh[:, c] for c in range(3)]
            return _dot(r, r) * (0.5 * m) - x[2] * (CLOTH_H**2 * GRAVITY[2] * m)
        return [(edges, spring), (torch.arange(nv, device=rest.device)[:, None], inertia)]

    # the learned density: features of the Green strain and of a second form from fixed vertex normals
    def normals(p):
        c = torch.linalg.cross(p[tris[:, 1]] - p[tris[:, 0]], p[tris[:, 2]] - p[tris[:, 0]])
        n = torch.zeros_like(p)
        for s in range(3):
            n.index_add_(0, tris[:, s], c)
        return n / n.norm(dim=1, keepdim=True)

    def second(a, b, nrm, k):
        n = [nrm[tris[k, s]] for s in range(3)]
        na = (n[1] - n[0]) * m00[k][:, None]
        nb = (n[1] - n[0]) * m01[k][:, None] + (n[2] - n[0]) * m11[k][:, None]
        na, nb = ([v[:, c] for c in range(3)] for v in (na, nb))
        return _dot(a, na) * -1.0, _dot(b, nb) * -1.0, (_dot(b, na) + _dot(a, nb)) * -0.5

    every = torch.arange(tris.shape[0], device=rest.device)
    ra, rb, *_ = strain([rest[tris[:, s], c] for s in range(3) for c in range(3)], every)
    rest_second, now = second(ra, rb, normals(rest), every), normals(d["x"])
    with np.load(mad.TRAINED_DENSITY, allow_pickle=False) as f:
        th = torch.from_numpy(f["theta"]).bfloat16().double().to(rest.device)   # the library evaluates BF16 weights
        s_in, s_out = torch.from_numpy(f["s_in"]).double().to(rest.device), float(f["s_out"][0])
    W1, b1, W2, b2, w3, b3 = (p.reshape(s) for p, s in zip(
        th.split([384, 64, 4096, 64, 64, 1]), ((64, 6), (64, 1), (64, 64), (64, 1), (64, 1), ())))
    sp = torch.nn.functional.softplus

    def learned(x, k):
        a, b, e0, e1, e2 = strain(x, k)
        z = [e0, e1, e2] + [p - q[k] for p, q in zip(second(a, b, now, k), rest_second)]
        zv = torch.stack([v.v for v in z]) * s_in[:, None]
        a1 = W1 @ zv + b1
        g1 = torch.sigmoid(a1)
        a2 = W2 @ sp(a1, threshold=100.0) + b2
        g2 = torch.sigmoid(a2)
        u = W2.t() @ (w3 * g2)
        T = [W2 @ (g1 * W1[:, i:i + 1]) for i in range(6)]
        first = [(s_out * s_in[i]) * (u * g1 * W1[:, i:i + 1]).sum(0) for i in range(6)]
        f = s_out * ((w3 * sp(a2, threshold=100.0)).sum(0) + b3)
        g = sum(first[i] * z[i].g for i in range(6))
        h = sum(first[i] * z[i].h for i in range(6))
        for i in range(6):
            for j in range(6):
                w = (u * g1 * (1 - g1) * W1[:, i:i + 1] * W1[:, j:j + 1]).sum(0)
                w = w + (w3 * g2 * (1 - g2) * T[i] * T[j]).sum(0)
                h = h + (s_out * s_in[i] * s_in[j] * w) * (z[i].g[:, None] * z[j].g[None])
        return _HD(f, g, h) * area[k]

    return [(tris, learned)]


def _exact_train(case, seed):
    d = {k: torch.from_numpy(v).double().cuda() if isinstance(v, np.ndarray) else v
         for k, v in _train_inputs(case, seed).items()}
    at = d["perm"][:case["n"]].long()
    z, W, dW, th = d["z"][at], d["W"][at], d["dW"][at], d["theta"].requires_grad_(True)
    W1, b1, W2, b2, w3, b3 = (p.reshape(s) for p, s in zip(
        th.split([384, 64, 4096, 64, 64, 1]), ((64, 6), (64,), (64, 64), (64,), (64,), ())))
    a1 = (z * d["s_in"]) @ W1.t() + b1
    h1, g1 = torch.log1p(torch.exp(-a1.abs())) + a1.clamp(min=0), torch.sigmoid(a1)
    a2 = h1 @ W2.t() + b2
    h2, g2 = torch.log1p(torch.exp(-a2.abs())) + a2.clamp(min=0), torch.sigmoid(a2)
    psi = d["s_out"] * (h2 @ w3 + b3)
    dpsi = d["s_out"] * d["s_in"] * (((g2 * w3) @ W2 * g1) @ W1)
    loss = (psi - W).square().mean() / d["c_e"] + ((dpsi - dW).square() / d["c_g"]).sum(1).mean()
    return torch.autograd.grad(loss, th)[0], loss.detach()[None]


def _exact_jacobian(d):
    tris, rest, x, vd = d["tris"].long(), d["rest"], d["x"], d["vdata"]
    edges = _edges(tris, rest.shape[0])[0]
    r = x[edges[:, 1]] - x[edges[:, 0]]
    length = r.norm(dim=1)
    k = math.sqrt(3.0)
    j = k * r / length[:, None]
    s = vd[:, 0].sqrt()
    res = torch.cat([k * (length - (rest[edges[:, 1]] - rest[edges[:, 0]]).norm(dim=1)),
                     (s[:, None] * (x - vd[:, 1:])).ravel()])
    eye = torch.eye(3, dtype=x.dtype, device=x.device)
    return res, torch.cat([torch.cat([-j, j], 1).ravel(), (s[:, None, None] * eye).ravel()])


def exact(case, seed):
    if case["ask"] == "train":
        return _exact_train(case, seed)
    d = {k: torch.from_numpy(v).cuda() if isinstance(v, np.ndarray) else v for k, v in _inputs(case, seed).items()}
    if case["ask"] == "jacobian":
        return _exact_jacobian(d)
    x, ask = d["x"], case["ask"]
    nv, dim = x.shape
    comp = d["comp"]
    terms = _terms(case, d)
    energy = torch.zeros(1 if comp is None else comp.numel(), dtype=torch.float64, device=x.device)
    grad, y = torch.zeros_like(x), torch.zeros_like(x)
    if ask in ("hess", "spd"):
        keys = [torch.arange(nv, device=x.device) * (nv + 1)]
        for st, _ in terms:
            for s in range(st.shape[1]):
                for t in range(s):
                    keys += [st[:, s] * nv + st[:, t], st[:, t] * nv + st[:, s]]
        keys = torch.unique(torch.cat(keys))
        hess = torch.zeros((keys.numel(), dim * dim), dtype=torch.float64, device=x.device)
    for st, f in terms:
        ns = st.shape[1]
        K = ns * dim
        for at in torch.arange(st.shape[0], device=x.device).split(200_000):
            sub = st[at]
            eye = torch.eye(K, dtype=x.dtype, device=x.device)
            zero = torch.zeros((1, 1, 1), dtype=x.dtype, device=x.device)
            e = f([_HD(x[sub[:, i // dim], i % dim], eye[:, i:i + 1], zero) for i in range(K)], at)
            g = e.g.expand(K, at.numel())
            where = 0 if comp is None else torch.searchsorted(comp, sub[:, 0].contiguous(), right=True) - 1
            if comp is None:
                energy[0] += e.v.sum()
            else:
                energy.index_add_(0, where + 1, e.v)
            for s in range(ns):
                grad.index_add_(0, sub[:, s], g[s * dim:(s + 1) * dim].t().contiguous())
            if ask == "grad":
                continue
            h = e.h.expand(K, K, at.numel())
            if ask in ("spd", "hvp"):
                h = _clamp(h)
            for s in range(ns):
                for t in range(ns):
                    b = h[s * dim:(s + 1) * dim, t * dim:(t + 1) * dim]
                    if ask == "hvp":
                        y.index_add_(0, sub[:, s], (b * d["v"][sub[:, t]].t()[None]).sum(1).t().contiguous())
                    else:
                        hess.index_add_(0, torch.searchsorted(keys, sub[:, s] * nv + sub[:, t]),
                                        b.reshape(dim * dim, -1).t().contiguous())
    if ask == "hvp":
        return y.ravel()
    if comp is not None:
        energy[0] = energy[1:].sum()
    if ask == "grad":
        return energy, grad.ravel()
    return energy, grad.ravel(), hess.reshape(-1, dim, dim)
