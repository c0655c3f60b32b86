"""Performance cases: the calls a user of the library makes, over their range of sizes.

A case is a dict of plain values.  ``listed()`` names the fixed ones, ``draw(rng)``
gives another one of the same ranges, ``prepare(case, seed)`` builds what a program
holds before the call (an uploaded Tucker handle, a dense plan, a geometry, device
buffers), ``run(state)`` is one call through the public entry points and returns its
outputs, ``exact(case, seed)`` the same outputs in 64 bits from plain torch, and
``work(case)`` the bytes and operations one call cannot do without.

Kinds of call
  pass    ``fmm_tucker_pass``: aggregation and disaggregation of all groups at once
  stages  ``fmm_tucker_aggregate``, then ``fmm_tucker_disaggregate``, as a solver calls
          them around its translation step
  dense   the plain method: ``fmm_dense_aggregate`` and ``fmm_dense_disaggregate``
  fill    the inputs of a problem from its mesh: ``fmm_farfield_fill`` of all groups and
          ``fmm_planewave_excitation``
  setup   a problem's compression: ``fmm_farfield_compress`` of a chunk of groups, the
          upload and one aggregation with the new factors

Shapes: a box edge of 0.5, 1, 1.5, 2 or 4 wavelengths fixes the angular grid, the mean
number of basis functions of a group and the mean multilinear ranks (the values of the
30-wavelength and 20-wavelength sphere workloads).  Group sizes are ragged, from a few
basis functions to about twice the mean, as a curved surface cuts its boxes.  Factors
have the scale of a compressed far-field: columns of about unit norm, a decaying core.
"""
import math
import random
import weakref

import numpy as np
import torch

import paper_2103_05822_amd as T

PREC = {"c128": T.FMM_C128, "c64": T.FMM_C64, "bf16x2": T.FMM_BF16X2, "bf16x3": T.FMM_BF16X3}

# box edge (wavelengths) -> n_theta, n_phi, mean n_beta, mean ranks (theta, phi, beta)
BOX = {
    0.5: (17, 33, 58, 15, 17, 47),
    1.0: (25, 49, 232, 18, 22, 93),
    1.5: (32, 63, 513, 22, 25, 132),
    2.0: (38, 75, 909, 23, 28, 167),
    4.0: (64, 127, 4408, 36, 50, 270),
}
# the small workload: a sphere of one wavelength, eight boxes of 0.5 on its own grid
SMALL = (14, 28, 240, 12, 18, 72)


def listed():
    return [
        # one iteration on the smallest problem, FP64: launches and latency count
        dict(name="small_c128_r1", kind="pass", box=0.0, prec="c128", nrhs=1, groups=8, grid=False, svd=False),
        # an iterative solver's pass with many small boxes
        dict(name="box05_c64_r1", kind="pass", box=0.5, prec="c64", nrhs=1, groups=2000, grid=False, svd=False),
        # the same with the paper's box size: the headline pass
        dict(name="box2_c64_r1", kind="pass", box=2.0, prec="c64", nrhs=1, groups=256, grid=False, svd=False),
        # FP64 stages onto the box grid of the FFT translation
        dict(name="box1_c128_r1_grid", kind="stages", box=1.0, prec="c128", nrhs=1, groups=400, grid=True, svd=False),
        # a handful of excitations at once, an odd number of them
        dict(name="box15_c64_r5", kind="pass", box=1.5, prec="c64", nrhs=5, groups=160, grid=False, svd=False),
        # monostatic sweeps: many plane waves per pass
        dict(name="box2_c64_r64", kind="pass", box=2.0, prec="c64", nrhs=64, groups=128, grid=False, svd=False),
        # the split precision with FP32 accuracy, as in the large workload
        dict(name="box2_bf16x3_r32", kind="pass", box=2.0, prec="bf16x3", nrhs=32, groups=128, grid=False, svd=False),
        # FP64 with several right-hand sides, stage by stage
        dict(name="box1_c128_r16", kind="stages", box=1.0, prec="c128", nrhs=16, groups=300, grid=False, svd=False),
        # the plain method, one right-hand side and eight
        dict(name="dense_box2_c128_r1", kind="dense", box=2.0, prec="c128", nrhs=1, groups=24),
        dict(name="dense_box1_c128_r8", kind="dense", box=1.0, prec="c128", nrhs=8, groups=200),
        # the inputs of a problem from its mesh
        dict(name="fill_plate64_box2", kind="fill", box=2.0, squares=64, nrhs=32),
        # compressing a chunk of groups
        dict(name="setup_plate20_box1", kind="setup", box=1.0, squares=20, digits=6),
    ]


# Budget of a drawn case, below the largest listed ones.
MAX_ELEMENTS = 1.2e8     # factor entries of a Tucker handle (memory and upload time)
MAX_FLOPS = 9.0e10       # Tucker passes
MAX_DENSE = 1.2e8        # dense far-field entries


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choices(["pass", "stages", "dense", "fill", "setup"], [50, 20, 15, 9, 6])[0]
    if kind == "fill":
        return dict(kind=kind, box=rng.choice([0.5, 1.0, 1.5, 2.0]), squares=_log_int(rng, 8, 64), nrhs=_log_int(rng, 1, 64))
    if kind == "setup":
        return dict(kind=kind, box=rng.choice([0.5, 1.0]), squares=_log_int(rng, 8, 20), digits=rng.choice([4, 5, 6]))
    if kind == "dense":
        box = rng.choice([0.5, 1.0, 1.5, 2.0])
        nt, npn, nb = BOX[box][:3]
        most = MAX_DENSE / (2.0 * nt * npn * nb)
        return dict(kind=kind, box=box, prec=rng.choice(["c128", "c128", "c64"]), nrhs=_log_int(rng, 1, 12),
                    groups=_log_int(rng, max(2, most / 64), max(3, most)))
    box = rng.choice([0.0, 0.5, 1.0, 1.5, 2.0, 2.0, 4.0])
    nt, npn, nb, rt, rp, rb = BOX[box] if box else SMALL
    prec = rng.choice(["c64", "c64", "c64", "c128", "c128", "bf16x3", "bf16x2"])
    nrhs = rng.choice([1, 1, _log_int(rng, 2, 64), _log_int(rng, 2, 64), 64])
    if prec.startswith("bf16"):
        nrhs += nrhs % 2
    svd = box in (0.5, 1.0) and rng.random() < 0.12
    if svd:
        rt, rp = nt, npn
    item = rb * (nb + rt * rp)
    flops = 32.0 * nrhs * (item + nt * rp * (rt + npn))  # both polarisations, both stages
    most = min(MAX_ELEMENTS / (2.0 * item), MAX_FLOPS / flops)
    groups = _log_int(rng, max(2, most / 64), max(3, most)) if box else rng.randint(4, 12)
    return dict(kind=kind, box=box, prec=prec, nrhs=nrhs, groups=min(groups, 2500), grid=rng.random() < 0.2, svd=svd)


# ------------------------------------------------------------------ Tucker cases

def _shapes(case):
    """Grid, offsets and the ranks [groups][2][3] of a Tucker or dense case: ragged, the
    same for every seed."""
    nt, npn, nbm, rtm, rpm, rbm = BOX[case["box"]] if case["box"] else SMALL
    rng = random.Random(1000 * case["groups"] + int(10 * case["box"]))
    nb, ranks = [], []
    for _ in range(case["groups"]):
        f = rng.uniform(0.03, 1.97)
        if not case["box"]:
            f = 1.0  # eight equal octants
        n = max(3, round(nbm * f))
        nb.append(n)
        pair = []
        for _ in range(2):
            if case.get("svd"):
                rt, rp = nt, npn
            else:
                rt = max(1, min(nt, n, round(rtm * f ** 0.1) + rng.randint(-2, 2)))
                rp = max(1, min(npn, n, round(rpm * f ** 0.1) + rng.randint(-2, 2)))
            rb = max(1, min(n, rt * rp, round(rbm * f ** 0.5) + rng.randint(-3, 3)))
            pair.append((rt, rp, rb))
        ranks.append(pair)
    offsets = np.concatenate([[0], np.cumsum(nb)]).astype(np.int64)
    return nt, npn, offsets, ranks


def _boxes(case):
    """A cubic box grid about three times the number of groups, and the groups' boxes."""
    k = max(2, math.ceil((3.0 * case["groups"]) ** (1.0 / 3.0)))
    boxes = sorted(random.Random(case["groups"]).sample(range(k ** 3), case["groups"]))
    return k, np.array(boxes, dtype=np.int64)


def _normal(gen, *shape, dtype=torch.complex64):
    """Circular complex Gaussian on the GPU; complex128 values are those of complex64."""
    return torch.randn(*shape, dtype=torch.complex64, device="cuda", generator=gen).to(dtype)


def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _factors(case, seed):
    """Factor blocks on the GPU per (group, polarisation), complex64: core, U^theta,
    U^phi, U^beta as views of one flat tensor, and that tensor.  Every value is a float,
    so that all precisions store it as it is."""
    nt, npn, off, ranks = _shapes(case)
    svd = case["svd"]
    sizes = []
    for g, pair in enumerate(ranks):
        n = int(off[g + 1] - off[g])
        for rt, rp, rb in pair:
            sizes.append((rt * rp * rb, 0 if svd else nt * rt, 0 if svd else npn * rp, n * rb))
    flat = _normal(_gen(seed), sum(map(sum, sizes)))
    at, items = 0, []
    for i, sz in enumerate(sizes):
        rt, rp, rb = ranks[i // 2][i % 2]
        n = int(off[i // 2 + 1] - off[i // 2])
        v = []
        for s in sz:
            v.append(flat[at:at + s])
            at += s
        core = v[0].view(rt, rp, rb)
        ramp = [torch.exp(torch.arange(m, device="cuda") * (-2.0 / m)) for m in (rt, rp, rb)]
        if svd:  # W = A conj(U^beta): only the basis mode decays
            core *= ramp[2] / math.sqrt(npn)
            ut = up = None
        else:
            core *= ramp[0][:, None, None] * ramp[1][None, :, None] * ramp[2]
            ut = v[1].view(nt, rt).mul_(1.0 / math.sqrt(nt))
            up = v[2].view(npn, rp).mul_(1.0 / math.sqrt(npn))
        items.append((core, ut, up, v[3].view(n, rb).mul_(1.0 / math.sqrt(n))))
    return items, flat


def _vec_dtype(case):
    return torch.complex128 if case["prec"] == "c128" else torch.complex64


def _tucker_vectors(case, seed, n_basis, n_dir):
    gen = _gen(seed + (1 << 40))
    rows = 2 * (_boxes(case)[0] ** 3 if case["grid"] else case["groups"])
    x = _normal(gen, n_basis, case["nrhs"], dtype=_vec_dtype(case))
    G = _normal(gen, rows, n_dir, case["nrhs"], dtype=_vec_dtype(case))
    return x, G


class _Held:
    """A library handle that is destroyed with the state that holds it."""

    def __init__(self, value, destroy):
        self.value = value
        self._f = weakref.finalize(self, destroy, value)


def _prepare_tucker(case, seed):
    nt, npn, off, ranks = _shapes(case)
    lay = T.Layout(nt, npn, off)
    items, flat = _factors(case, seed)
    host = flat.to(torch.complex128).cpu().numpy()
    h = T.fmm_tucker_create(lay)
    held = _Held(h, T.fmm_tucker_destroy)
    eye_t, eye_p = np.eye(nt, dtype=np.complex128), np.eye(npn, dtype=np.complex128)
    at = 0
    for i, (core, ut, up, ub) in enumerate(items):
        v = []
        for t in (core, ut, up, ub):
            if t is None:
                v.append(None)
                continue
            v.append(host[at:at + t.numel()].reshape(tuple(t.shape)))
            at += t.numel()
        T.fmm_tucker_set_group(h, i // 2, i % 2, v[0], eye_t if v[1] is None else v[1], eye_p if v[2] is None else v[2], v[3])
    if case["grid"]:
        k, boxes = _boxes(case)
        T.fmm_tucker_set_box_grid(h, (k, k, k), boxes)
    prec = PREC[case["prec"]]
    arena = torch.empty(T.fmm_tucker_storage_bytes(h, prec)[1], dtype=torch.uint8, device="cuda")
    T.fmm_tucker_upload(h, prec, arena)
    x, G = _tucker_vectors(case, seed, int(off[-1]), nt * npn)
    return dict(kind=case["kind"], handle=held, arena=arena, prec=prec, nrhs=case["nrhs"], x=x, G=G,
                F=torch.empty_like(G), V=torch.empty_like(x))


def _exact_tucker(case, seed):
    nt, npn, off, ranks = _shapes(case)
    items, _ = _factors(case, seed)
    x, G = _tucker_vectors(case, seed, int(off[-1]), nt * npn)
    R = case["nrhs"]
    x, G = x.to(torch.complex128), G.to(torch.complex128)
    F, V = torch.zeros_like(G), torch.zeros_like(x)
    k, boxes = _boxes(case) if case["grid"] else (0, None)
    for i, f in enumerate(items):
        core, ut, up, ub = (t if t is None else t.to(torch.complex128) for t in f)
        rt, rp, rb = core.shape
        g, a = divmod(i, 2)
        rows = slice(int(off[g]), int(off[g + 1]))
        fibre = 2 * g + a if boxes is None else a * k ** 3 + int(boxes[g])
        core = core.reshape(rt * rp, rb)
        t = core @ (ub.T.contiguous() @ x[rows])
        s = G[fibre].conj().resolve_conj()
        if ut is not None:
            t = (ut @ t.reshape(rt, rp * R)).reshape(nt, rp, R).permute(1, 0, 2).reshape(rp, nt * R)
            t = (up @ t).reshape(npn, nt, R).permute(1, 0, 2).reshape(nt * npn, R)
            s = (ut.T.contiguous() @ s.reshape(nt, npn * R)).reshape(rt, npn, R).permute(1, 0, 2).reshape(npn, rt * R)
            s = (up.T.contiguous() @ s).reshape(rp, rt, R).permute(1, 0, 2).reshape(rt * rp, R)
        F[fibre] = t
        V[rows] += (ub @ (core.T.contiguous() @ s)).conj()
    return F, V


def _work_tucker(case):
    nt, npn, off, ranks = _shapes(case)
    es, R, nd = (16 if case["prec"] == "c128" else 8), case["nrhs"], nt * npn
    factors = flops = 0
    for g, pair in enumerate(ranks):
        n = int(off[g + 1] - off[g])
        for rt, rp, rb in pair:
            big = rb * (n + rt * rp)
            ang = 0 if case["svd"] else min(nt * rp * (rt + npn), rt * npn * (rp + nt))
            factors += big + (0 if case["svd"] else nt * rt + npn * rp)
            flops += 2 * 8 * R * (big + ang)
    n_items = 2 * len(ranks)
    grid = 2 * _boxes(case)[0] ** 3 if case["grid"] else n_items
    factors *= 2 if case["kind"] == "stages" else 1  # two calls, each of which reads them once
    vectors = R * (2 * int(off[-1]) + nd * (n_items + grid))
    return {"bytes": es * (factors + vectors), "flops": flops}


# ------------------------------------------------------------------- dense cases

def _dense_inputs(case, seed):
    nt, npn, off, _ = _shapes(case)
    gen, dt, n = _gen(seed), _vec_dtype(case), int(off[-1])
    A = torch.empty(n, 2, nt * npn, dtype=dt, device="cuda")
    for r in range(0, n, 4096):
        A[r:r + 4096] = _normal(gen, min(4096, n - r), 2, nt * npn, dtype=dt)
    x = _normal(gen, n, case["nrhs"], dtype=dt)
    G = _normal(gen, case["groups"], 2 * nt * npn, case["nrhs"], dtype=dt)
    return nt, npn, off, A, x, G


def _prepare_dense(case, seed):
    nt, npn, off, A, x, G = _dense_inputs(case, seed)
    plan = _Held(T.fmm_dense_create(T.Layout(nt, npn, off)), T.fmm_dense_destroy)
    return dict(kind="dense", plan=plan, prec=PREC[case["prec"]], nrhs=case["nrhs"], A=A, x=x, G=G,
                F=torch.empty_like(G), V=torch.empty_like(x))


def _exact_dense(case, seed):
    nt, npn, off, A, x, G = _dense_inputs(case, seed)
    z = torch.complex128
    x, G = x.to(z), G.to(z)
    F, V = torch.empty_like(G), torch.empty_like(x)
    for g in range(case["groups"]):
        rows = slice(int(off[g]), int(off[g + 1]))
        a = A[rows].reshape(-1, 2 * nt * npn).to(z)
        F[g] = a.T.contiguous() @ x[rows]
        V[rows] = a.conj().resolve_conj() @ G[g]
    return F, V


def _work_dense(case):
    nt, npn, off, _ = _shapes(case)
    es, R, n, nd = (16 if case["prec"] == "c128" else 8), case["nrhs"], int(off[-1]), 2 * nt * npn
    # the far-fields serve two calls, each of which reads them once
    return {"bytes": es * (2 * n * nd + 2 * R * (n + case["groups"] * nd)), "flops": 16 * R * n * nd}


# ------------------------------------------------------- cases that start from a mesh

K_WAVE = 2.0 * math.pi


def _plate(case, seed):
    """A gently curved plate of squares x squares cells, a tenth of a wavelength each, two
    triangles per cell, in one layer of boxes; the seed changes its curvature."""
    n = case["squares"]
    a, b, c = np.random.default_rng(seed).uniform(0.5, 1.5, 3)
    u, v = np.meshgrid(np.arange(n + 1) * 0.1, np.arange(n + 1) * 0.1, indexing="ij")
    z = 0.12 * np.sin(a * u + b) + 0.1 * np.cos(c * v)
    verts = np.stack([u, v, z], axis=-1).reshape(-1, 3)
    i, j = np.meshgrid(np.arange(n), np.arange(n), indexing="ij")
    p = (i * (n + 1) + j).reshape(-1)
    q = p + n + 1
    tris = np.concatenate([np.stack([p, q, q + 1], 1), np.stack([p, q + 1, p + 1], 1)]).astype(np.int32)
    origin = np.array([-0.0123, -0.0171, -0.5 * case["box"]])
    return verts, tris, origin, math.ceil((0.1 * n + 0.02) / case["box"])


def _waves(case, seed):
    gen = np.random.default_rng(seed + 7)
    k = gen.standard_normal((case["nrhs"], 3))
    k /= np.linalg.norm(k, axis=1, keepdims=True)
    e = np.cross(k, gen.standard_normal((case["nrhs"], 3)))
    return k, e / np.linalg.norm(e, axis=1, keepdims=True)


def _geometry(case, seed):
    verts, tris, origin, per_axis = _plate(case, seed)
    nt, npn = BOX[case["box"]][:2]
    return T.fmm_geometry_build(verts, tris, origin, case["box"], per_axis, K_WAVE, nt, npn)


def _prepare_fill(case, seed):
    geom = _Held(_geometry(case, seed), T.fmm_geometry_destroy)
    lay = T.fmm_geometry_layout(geom.value)
    ff = torch.empty(lay.n_basis, 2, lay.n_theta, lay.n_phi, dtype=torch.complex128, device="cuda")
    x = torch.empty(lay.n_basis, case["nrhs"], dtype=torch.complex128, device="cuda")
    T.fmm_farfield_fill(geom.value, 0, 1, ff)  # the geometry is on the device from its first call on
    k, e = _waves(case, seed)
    return dict(kind="fill", geom=geom, groups=lay.n_groups, ff=ff, x=x, khat=k, epol=e)


def _rows(case, seed):
    """Points [N, 6, 3], weighted RWG vectors [N, 6, 3] and box centres [N, 3] of the
    3-point rule on both triangles of every basis function, in group order."""
    verts, tris, origin, K = _plate(case, seed)
    t = tris.astype(np.int64)
    u, w, o = t.reshape(-1), t[:, [1, 2, 0]].reshape(-1), t[:, [2, 0, 1]].reshape(-1)
    tri = np.repeat(np.arange(len(t)), 3)
    lo, hi = np.minimum(u, w), np.maximum(u, w)
    order = np.lexsort((u > w, hi, lo))  # per edge: the triangle traversing lo -> hi first
    lo, hi, o, tri = lo[order], hi[order], o[order], tri[order]
    first = np.flatnonzero((lo[1:] == lo[:-1]) & (hi[1:] == hi[:-1]))
    mid = 0.5 * (verts[lo[first]] + verts[hi[first]])
    idx = np.clip(np.floor((mid - origin) / case["box"]), 0, K - 1).astype(np.int64)
    first = first[np.argsort((idx[:, 0] * K + idx[:, 1]) * K + idx[:, 2], kind="stable")]
    mid = 0.5 * (verts[lo[first]] + verts[hi[first]])
    idx = np.clip(np.floor((mid - origin) / case["box"]), 0, K - 1)
    length = np.linalg.norm(verts[hi[first]] - verts[lo[first]], axis=1)
    B = np.array([[4.0, 1.0, 1.0], [1.0, 4.0, 1.0], [1.0, 1.0, 4.0]]) / 6.0
    pts, rho = [], []
    for side, sign in ((0, 1.0), (1, -1.0)):
        r = np.einsum("qk,nkc->nqc", B, verts[t[tri[first + side]]])
        pts.append(r)
        rho.append(sign * (r - verts[o[first + side]][:, None, :]) * (length / 6.0)[:, None, None])
    return np.concatenate(pts, 1), np.concatenate(rho, 1), origin + (idx + 0.5) * case["box"]


def _directions(case):
    """(k, theta, phi unit vectors) [n_dir, 3] of the grid: Gauss-Legendre in cos(theta),
    theta increasing, phi uniform."""
    nt, npn = BOX[case["box"]][:2]
    th = np.arccos(np.polynomial.legendre.leggauss(nt)[0][::-1])
    st, ct = np.sin(th)[:, None], np.cos(th)[:, None]
    ph = 2.0 * np.pi * np.arange(npn) / npn
    sp, cp = np.sin(ph)[None], np.cos(ph)[None]
    one = np.ones((nt, npn))
    vec = lambda a, b, c: torch.from_numpy(np.stack([a * one, b * one, c * one], -1).reshape(-1, 3)).cuda()  # noqa: E731
    return vec(st * cp, st * sp, ct), vec(ct * cp, ct * sp, -st), vec(-sp, cp, 0.0)


def _exact_fill(case, seed):
    pts, rho, c = (torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in _rows(case, seed))
    k, th, ph = _directions(case)
    n, nd = pts.shape[0], k.shape[0]
    ff = torch.empty(n, 2, nd, dtype=torch.complex128, device="cuda")
    rel = pts - c[:, None, :]
    for r in range(0, n, 512):
        e = torch.zeros(2, min(512, n - r), nd, dtype=torch.complex128, device="cuda")
        for q in range(6):
            w = torch.polar(torch.ones((), dtype=torch.float64, device="cuda"), K_WAVE * (rel[r:r + 512, q] @ k.T))
            e[0] += (rho[r:r + 512, q] @ th.T) * w
            e[1] += (rho[r:r + 512, q] @ ph.T) * w
        ff[r:r + 512] = e.transpose(0, 1)
    kh, ep = (torch.from_numpy(a).cuda() for a in _waves(case, seed))
    x = torch.zeros(n, case["nrhs"], dtype=torch.complex128, device="cuda")
    for q in range(6):
        x -= (rho[:, q] @ ep.T) * torch.polar(torch.ones((), dtype=torch.float64, device="cuda"), -K_WAVE * (pts[:, q] @ kh.T))
    nt, npn = BOX[case["box"]][:2]
    return ff.view(n, 2, nt, npn), x


def _mesh_rows(case):
    n = case["squares"]
    return 3 * n * n - 2 * n


def _work_fill(case):
    n, nd = _mesh_rows(case), BOX[case["box"]][0] * BOX[case["box"]][1]
    # per point and direction or wave: the phase (6), its sine and cosine (about 40 with
    # a short polynomial each) and the weighted sums
    return {"bytes": n * (16 * (2 * nd + case["nrhs"]) + 8 * 37),
            "flops": n * 6 * (nd * (6 + 40 + 20) + case["nrhs"] * (6 + 40 + 10))}


def _prepare_setup(case, seed):
    geom = _Held(_geometry(case, seed), T.fmm_geometry_destroy)
    lay = T.fmm_geometry_layout(geom.value)
    ff = torch.empty(lay.n_basis, 2, lay.n_theta, lay.n_phi, dtype=torch.complex128, device="cuda")
    T.fmm_farfield_fill(geom.value, 0, lay.n_groups, ff)
    x = _normal(_gen(seed), lay.n_basis, 1, dtype=torch.complex128)
    F = torch.empty(lay.n_groups, 2, lay.n_dir, 1, dtype=torch.complex128, device="cuda")
    return dict(kind="setup", layout=lay, gamma=10.0 ** -case["digits"], ff=ff, x=x, F=F)


def _run_setup(s):
    h = T.fmm_farfield_compress(s["layout"], s["ff"], 0, s["layout"].n_groups, s["gamma"])
    arena = torch.empty(T.fmm_tucker_storage_bytes(h, T.FMM_C128)[1], dtype=torch.uint8, device="cuda")
    T.fmm_tucker_upload(h, T.FMM_C128, arena)
    T.fmm_tucker_aggregate(h, T.FMM_C128, 1, s["x"], s["F"])
    ranks = T.fmm_tucker_ranks(h, s["layout"].n_groups)
    torch.cuda.current_stream().synchronize()  # the arena and the handle go out of use here
    T.fmm_tucker_destroy(h)
    return s["F"], ranks


def _work_setup(case):
    nt, npn, nb = BOX[case["box"]][:3]
    n, nd, g = _mesh_rows(case), nt * npn, max(1.0, (0.1 * case["squares"] / case["box"]) ** 2)
    m = n / g  # basis functions of a group: two Gram products and an eigensolution (about
    # nine m^3 complex operations) per polarisation
    return {"bytes": 16 * 2 * n * nd, "flops": 2 * g * 8 * (m * m * nd + m * nd * (nt + npn) + 9 * m ** 3)}


# --------------------------------------------------------------------------------

def prepare(case, seed):
    how = {"pass": _prepare_tucker, "stages": _prepare_tucker, "dense": _prepare_dense, "fill": _prepare_fill, "setup": _prepare_setup}
    return how[case["kind"]](case, seed)


def run(s):
    kind = s["kind"]
    if kind == "pass":
        T.fmm_tucker_pass(s["handle"].value, s["prec"], s["nrhs"], s["x"], s["F"], s["G"], s["V"])
    elif kind == "stages":
        T.fmm_tucker_aggregate(s["handle"].value, s["prec"], s["nrhs"], s["x"], s["F"])
        T.fmm_tucker_disaggregate(s["handle"].value, s["prec"], s["nrhs"], s["G"], s["V"])
    elif kind == "dense":
        T.fmm_dense_aggregate(s["plan"].value, s["prec"], s["A"], s["nrhs"], s["x"], s["F"])
        T.fmm_dense_disaggregate(s["plan"].value, s["prec"], s["A"], s["nrhs"], s["G"], s["V"])
    elif kind == "fill":
        T.fmm_farfield_fill(s["geom"].value, 0, s["groups"], s["ff"])
        T.fmm_planewave_excitation(s["geom"].value, s["khat"], s["epol"], T.FMM_C128, s["x"])
        return s["ff"], s["x"]
    else:
        return _run_setup(s)
    return s["F"], s["V"]


def exact(case, seed):
    how = {"pass": _exact_tucker, "stages": _exact_tucker, "dense": _exact_dense, "fill": _exact_fill}
    if case["kind"] == "setup":
        return None  # the ranks and the spectra of a truncated decomposition: no value but its own
    return how[case["kind"]](case, seed)


def work(case):
    how = {"pass": _work_tucker, "stages": _work_tucker, "dense": _work_dense, "fill": _work_fill, "setup": _work_setup}
    return how[case["kind"]](case)
