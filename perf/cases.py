"""Performance cases of the level-set evaluator: what a program that smooths
triangulated solids has it do, from one small evaluation to the build and
evaluation of a two-million-triangle skeleton.

A case is a dict of plain values; its "kind" names the call:

  eval         Phi and grad Phi at given targets through lss_eval, by every
               pair or through the octree; with "step" the width is set anew
               and the octree rebuilt in the pass (the widths of a skeleton are
               changed and the field evaluated again), without it the context
               is built beforehand and only queried
  noalloc      the same query through the allocation-free entry point
  project      Newton projection of the chart nodes of every triangle, after
               a change of the widths, or from a new skeleton ("fresh")
  batch        a ragged batch of meshes in one context: new widths, the field
               at each mesh's own targets, and the charts of every mesh
  post         tangents, area element, normals, second derivatives and
               curvatures of projected charts
  multiscale   Phi, grad Phi and sigma(x) with the target-attached width
  interp       interpolation of chart data from the chart nodes to other
               points of every triangle

Sizes are those of the repository's workloads (the 3072-triangle cube with
4096 targets, the 20 480-triangle sphere with up to 1e6, the 2e5-triangle
graded surface with 45 chart nodes per triangle, the ragged batch of star
surfaces with 500 triangles and more each, the 2e6-triangle graded sphere with
5e7 targets), of its refinement study (hundreds to thousands of triangles, 15
or 45 chart nodes) and in between.  The skeletons here are cube grids mapped to
a cube, a sphere or a star-shaped surface with seeded waves, graded by a
conformal map where the case says so; they are made on the GPU.
"""
import math

import numpy as np
import torch

import paper_1909_13356_amd as lss

DEV = "cuda"
CUT = {True: math.sqrt(40.0), False: 8.0}        # near radius in units of sigma: mixed, FP64


# ------------------------------------------------------------------ cases
def listed():
    return [
        # one query of a small solid by the exact sum: the 3072-triangle cube and its 4096 targets
        dict(name="cube-direct-fp64", kind="eval", mesh="cube", n=16, grade=1.0, mixed=False, fmm=False, step=False,
             targets=4096, where="box"),
        # a serving loop's small query of a skeleton that is already built
        dict(name="sphere-query-noalloc-mixed", kind="noalloc", mesh="sphere", n=41, grade=1.0, mixed=True, fmm=True,
             step=False, targets=1000, where="near"),
        # the exact sum as a workhorse: 2e4 triangles, a quarter of a million targets around the surface
        dict(name="sphere-direct-mixed", kind="eval", mesh="sphere", n=41, grade=1.0, mixed=True, fmm=False,
             step=False, targets=250_001, where="shell"),
        # a refinement study's unit of work: a new skeleton of a few thousand triangles, its order-8 charts
        dict(name="charts-new-skeleton-fp64", kind="project", mesh="star", n=12, grade=1.0, mixed=False, nodes=45,
             fresh=True),
        # charts at order 4 (15 nodes) in FP64 after a change of the widths, 3e4 triangles
        dict(name="charts-fp64", kind="project", mesh="star", n=51, grade=3.0, mixed=False, nodes=15, fresh=False),
        # the graded 2e5-triangle surface and its 9e6 order-8 chart nodes, mixed
        dict(name="charts-graded-mixed", kind="project", mesh="star", n=129, grade=10.0, mixed=True, nodes=45,
             fresh=False),
        # new widths, build and field in FP64: 2e5 triangles, 2e6 targets near the surface
        dict(name="step-graded-fp64", kind="eval", mesh="star", n=129, grade=10.0, mixed=False, fmm=True, step=True,
             targets=2_000_003, where="near"),
        # the largest: new widths, build and field, 2e6 triangles, 5e7 targets near the surface
        dict(name="step-large-mixed", kind="eval", mesh="star", n=408, grade=10.0, mixed=True, fmm=True, step=True,
             targets=50_000_000, where="near"),
        # a ragged batch of star surfaces in one context: field at 2000 targets each, and every chart
        dict(name="batch-mixed", kind="batch", mixed=True, surfaces=24, nmin=7, nmax=33, targets=2000, nodes=15),
        # what follows a projection: tangents, normals and curvatures of 3e5 charts' nodes
        dict(name="curvature-fp64", kind="post", mesh="star", n=23, grade=2.0, mixed=False, nodes=45),
        # the target-attached width at 1e5 points of a graded surface
        dict(name="multiscale-mixed", kind="multiscale", mesh="star", n=60, grade=3.0, mixed=True, targets=100_000,
             where="near"),
        # chart data of 2e5 triangles carried to other points: 45 -> 66 nodes, three components
        dict(name="interp-charts", kind="interp", n=129, nodes=45, points=66, comps=3),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["eval", "eval", "eval", "noalloc", "project", "project", "batch", "post", "multiscale",
                       "interp"])
    mixed = rng.random() < 0.5
    if kind == "eval":
        if rng.random() < 0.4:                       # every pair: small solids, or some targets of a larger one
            n = _log(rng, 8, 41)
            return dict(kind=kind, mesh=rng.choice(["cube", "sphere", "star"]), n=n, grade=1.0, mixed=mixed,
                        fmm=False, step=False, targets=_log(rng, 500, 250_001), where=rng.choice(["box", "shell"]))
        n = _log(rng, 20, 300)
        return dict(kind=kind, mesh="star", n=n, grade=round(rng.uniform(1.0, 10.0), 2), mixed=mixed, fmm=True,
                    step=rng.random() < 0.7, targets=_log(rng, 5_000, 10_000_000 if mixed else 3_000_000),
                    where=rng.choice(["near", "near", "shell"]))
    if kind == "noalloc":
        return dict(kind=kind, mesh=rng.choice(["sphere", "star"]), n=_log(rng, 12, 129), grade=1.0, mixed=mixed,
                    fmm=rng.random() < 0.8, step=False, targets=_log(rng, 64, 20_000), where="near")
    if kind == "project":
        fresh = rng.random() < 0.5
        return dict(kind=kind, mesh="star", n=_log(rng, 6, 24 if fresh else 100),
                    grade=round(rng.uniform(1.0, 2.0 if fresh else 8.0), 2), mixed=mixed,
                    nodes=rng.choice([15, 28, 45]), fresh=fresh)
    if kind == "batch":
        return dict(kind=kind, mixed=mixed, surfaces=rng.randint(3, 40), nmin=7, nmax=_log(rng, 10, 33),
                    targets=_log(rng, 200, 10_000), nodes=rng.choice([15, 45]))
    if kind == "post":
        return dict(kind=kind, mesh="star", n=_log(rng, 10, 60), grade=round(rng.uniform(1.0, 4.0), 2), mixed=mixed,
                    nodes=rng.choice([15, 45]))
    if kind == "multiscale":
        return dict(kind=kind, mesh="star", n=_log(rng, 16, 100), grade=round(rng.uniform(1.0, 4.0), 2), mixed=mixed,
                    targets=_log(rng, 3_000, 300_000), where=rng.choice(["near", "shell"]))
    return dict(kind="interp", n=_log(rng, 12, 129), nodes=rng.choice([15, 28, 45]), points=rng.choice([10, 36, 66]),
                comps=rng.choice([1, 3]))


# -------------------------------------------------------------- skeletons
def dunavant6():
    """Dunavant's 12-node degree-6 rule on the unit triangle: rows (u, v, w)."""
    rows = []
    for a, w in ((0.249286745170910421, 0.116786275726379366), (0.063089014491502228, 0.050844906370206817)):
        b = 1.0 - 2.0 * a
        rows += [(u, v, 0.5 * w) for u, v in ((a, a), (a, b), (b, a))]
    b, c, w = 0.053145049844816947, 0.310352451033784405, 0.082851075618373575
    d = 1.0 - b - c
    rows += [(u, v, 0.5 * w) for u, v in ((b, c), (c, b), (b, d), (d, b), (c, d), (d, c))]
    return np.array(rows)


def chart_nodes(count):
    """The `count` = (p + 1)(p + 2) / 2 interior lattice nodes of order p on the unit triangle."""
    p = round((math.sqrt(8 * count + 1) - 3) / 2)
    return np.array([((i + 1) / (p + 3), (j + 1) / (p + 3)) for j in range(p + 1) for i in range(p + 1 - j)])


def cube_grid(n):
    """Vertices (integers 0..n) and outward triangles of the surface of an n x n x n cube grid."""
    r = torch.arange(n, device=DEV)
    i, j = (t.reshape(-1) for t in torch.meshgrid(r, r, indexing="ij"))
    quads = []
    for axis in range(3):
        u, v = (axis + 1) % 3, (axis + 2) % 3
        for side in (0, n):
            corner = []
            for du, dv in ((0, 0), (1, 0), (1, 1), (0, 1)):
                p = torch.empty((len(i), 3), dtype=torch.int64, device=DEV)
                p[:, axis], p[:, u], p[:, v] = side, i + du, j + dv
                corner.append((p[:, 0] * (n + 1) + p[:, 1]) * (n + 1) + p[:, 2])
            quads.append(corner if side else corner[::-1])
    a, b, c, d = (torch.cat([q[k] for q in quads]) for k in range(4))
    tris = torch.cat([torch.stack([a, b, c], 1), torch.stack([a, c, d], 1)])
    code, tris = torch.unique(tris, return_inverse=True)
    verts = torch.stack([code // ((n + 1) * (n + 1)), code // (n + 1) % (n + 1), code % (n + 1)], 1)
    return verts.double(), tris.to(torch.int32).contiguous()


def diameters(verts, tris):
    """Diameter of the smallest ball enclosing each triangle."""
    p = verts[tris.long()]
    e = torch.stack([(p[:, 1] - p[:, 2]).square().sum(1), (p[:, 2] - p[:, 0]).square().sum(1),
                     (p[:, 0] - p[:, 1]).square().sum(1)], 1)
    area2 = torch.linalg.cross(p[:, 1] - p[:, 0], p[:, 2] - p[:, 0]).norm(dim=1)
    most = e.max(1).values
    return torch.where(2.0 * most >= e.sum(1), most.sqrt(), e.prod(1).sqrt() / area2)


def skeleton(mesh, n, grade, g):
    """(verts, tris, sigma) of a closed surface with 12 n^2 triangles: the unit cube with sigma 0.1, the unit sphere
    with sigma 0.05 (both on a plain grid), or a star-shaped surface with seeded waves and bumps, graded by the
    conformal dilation `grade` (edge lengths spread over grade^2), with sigma half the triangle's diameter."""
    verts, tris = cube_grid(n)
    if mesh == "cube":
        shift = 0.01 * torch.rand(3, generator=g, dtype=torch.float64, device=DEV)
        return verts / n + shift, tris, torch.full((1,), 0.1, dtype=torch.float64, device=DEV)
    q = torch.tan((verts / n - 0.5) * (0.5 * math.pi))
    q = q / q.norm(dim=1, keepdim=True)
    if grade != 1.0:                                 # stereographic dilation of the sphere
        s = (1.0 + q[:, 2]) + grade * grade * (1.0 - q[:, 2])
        q = torch.cat([2.0 * grade * q[:, :2] / s[:, None],
                       (((1.0 + q[:, 2]) - grade * grade * (1.0 - q[:, 2])) / s)[:, None]], 1)
        q = q / q.norm(dim=1, keepdim=True)
    if mesh == "sphere":
        turn, _ = torch.linalg.qr(torch.randn((3, 3), generator=g, dtype=torch.float64, device=DEV))
        turn = turn * torch.sign(torch.linalg.det(turn))
        return (q @ turn).contiguous(), tris, torch.full((1,), 0.05, dtype=torch.float64, device=DEV)
    k = torch.randn((24, 3), generator=g, dtype=torch.float64, device=DEV) * 2.0
    ph = torch.rand(24, generator=g, dtype=torch.float64, device=DEV) * (2.0 * math.pi)
    r = 1.0 + 0.02 * torch.cos(q @ k.T + ph).sum(1)
    c = torch.randn((40, 3), generator=g, dtype=torch.float64, device=DEV)
    c = c / c.norm(dim=1, keepdim=True)
    w = 0.15 + 0.25 * torch.rand(40, generator=g, dtype=torch.float64, device=DEV)
    h = 0.03 * (2.0 * torch.rand(40, generator=g, dtype=torch.float64, device=DEV) - 1.0)
    for b in range(40):
        r = r + h[b] * torch.exp(-(q - c[b]).square().sum(1) / (2.0 * w[b] * w[b]))
    verts = (q * r[:, None]).contiguous()
    return verts, tris, (0.5 * diameters(verts, tris)).contiguous()


def points(where, count, verts, tris, sigma, g):
    """Targets: in a box twice the solid's size, in a shell around the unit sphere, or near the surface (a uniform
    surface point offset by t sigma along the normal, t in [-3, 3]: the spread of Newton iterates)."""
    f = dict(generator=g, dtype=torch.float64, device=DEV)
    if where == "box":
        lo, hi = verts.min(0).values, verts.max(0).values
        return lo - 0.5 * (hi - lo) + 2.0 * (hi - lo) * torch.rand((count, 3), **f)
    if where == "shell":
        d = torch.randn((count, 3), **f)
        return d / d.norm(dim=1, keepdim=True) * (0.5 + torch.rand((count, 1), **f))
    p = verts[tris.long()]
    nrm = torch.linalg.cross(p[:, 1] - p[:, 0], p[:, 2] - p[:, 0])
    area2 = nrm.norm(dim=1)
    cdf = torch.cumsum(area2, 0)
    j = torch.searchsorted(cdf, torch.rand(count, **f) * cdf[-1]).clamp_(max=len(tris) - 1)
    uv = torch.rand((count, 2), **f)
    uv = torch.where(uv.sum(1, keepdim=True) > 1.0, 1.0 - uv, uv)
    t = 6.0 * torch.rand(count, **f) - 3.0
    t = t * sigma[j if len(sigma) > 1 else torch.zeros_like(j)] / area2[j]
    x = torch.empty((count, 3), dtype=torch.float64, device=DEV)
    for a in range(0, count, 1 << 23):               # the largest case has 5e7 targets
        s = slice(a, a + (1 << 23))
        q = p[j[s]]
        x[s] = q[:, 0] + uv[s, :1] * (q[:, 1] - q[:, 0]) + uv[s, 1:] * (q[:, 2] - q[:, 0]) + t[s, None] * nrm[j[s]]
    return x


def batch_skeletons(case, g):
    """The meshes of a ragged batch as one vertex / triangle array with offsets, and each mesh's targets."""
    vs, ts, ss, xs, off, nv = [], [], [], [], [0], 0
    for m in range(case["surfaces"]):                # triangle counts log-uniform, in no order of size
        u = (m * 0.6180339887498949) % 1.0
        n = int(round(case["nmin"] * (case["nmax"] / case["nmin"]) ** u))
        v, t, s = skeleton("star", n, 1.0, g)
        xs.append(points("box", case["targets"], v, t, s, g))
        vs.append(v)
        ts.append(t + nv)
        ss.append(s)
        nv += len(v)
        off.append(off[-1] + len(t))
    xm = torch.arange(case["surfaces"], dtype=torch.int32, device=DEV).repeat_interleave(case["targets"])
    return (torch.cat(vs), torch.cat(ts).contiguous(), torch.cat(ss), torch.tensor(off, device=DEV),
            torch.cat(xs), xm)


def generator(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def inputs(case, seed):
    """Everything that a case's calls read, from the seed alone."""
    g, kind, s = generator(seed), case["kind"], {}
    if kind == "batch":
        s["verts"], s["tris"], s["sigma"], s["off"], s["x"], s["xm"] = batch_skeletons(case, g)
    else:
        s["verts"], s["tris"], s["sigma"] = skeleton(case.get("mesh", "star"), case["n"], case.get("grade", 1.0), g)
        if "targets" in case:
            s["x"] = points(case["where"], case["targets"], s["verts"], s["tris"], s["sigma"], g)
    if "nodes" in case:
        s["uv"] = torch.tensor(chart_nodes(case["nodes"]), device=DEV)
    if kind == "interp":
        s["data"] = torch.randn((len(s["tris"]) * case["nodes"], case["comps"]), generator=g, dtype=torch.float64,
                                device=DEV)
        s["to"] = torch.tensor(chart_nodes(case["points"]), device=DEV)
    return s


# ------------------------------------------------------------------- pass
def prepare(case, seed):
    s = inputs(case, seed)
    s["kind"], s["case"] = case["kind"], case
    s["rule"] = torch.tensor(dunavant6(), device=DEV)
    ctx = s["ctx"] = lss.Context()
    fmm = case.get("fmm", True)
    ctx.set_options(precision=lss.MIXED if case.get("mixed") else lss.FP64,
                    far_field=lss.FAR_FMM if fmm else lss.FAR_DIRECT)
    if case.get("fresh"):
        return s                                     # the pass brings the skeleton
    ctx.set_sources(s["verts"], s["tris"], s["rule"], tri_offsets=s.get("off"))
    ctx.set_sigma(s["sigma"])
    if case["kind"] in ("eval", "noalloc", "post") and not case.get("step"):
        ctx.build()
    if case["kind"] == "noalloc":                    # a serving loop keeps its output buffers
        s["phi"] = torch.empty(len(s["x"]), dtype=torch.float64, device=DEV)
        s["grad"] = torch.empty((len(s["x"]), 3), dtype=torch.float64, device=DEV)
    if case["kind"] == "post":
        s["h"] = ctx.project(s["uv"], device=True)[0]
    return s


def run(s):
    ctx, case = s["ctx"], s["case"]
    if s["kind"] == "eval":
        if case["step"]:
            ctx.set_sigma(s["sigma"])
        return ctx.eval(s["x"])
    if s["kind"] == "noalloc":
        return ctx.eval_noalloc(s["x"], s["phi"], s["grad"])
    if s["kind"] == "project":
        if case["fresh"]:
            ctx.set_sources(s["verts"], s["tris"], s["rule"])
        ctx.set_sigma(s["sigma"])
        return ctx.project(s["uv"], device=True)[:3]     # h, x, status (iters is a diagnostic)
    if s["kind"] == "batch":
        ctx.set_sigma(s["sigma"])
        phi, grad = ctx.eval(s["x"], x_mesh=s["xm"])
        return (phi, grad) + tuple(ctx.project(s["uv"], device=True)[:3])
    if s["kind"] == "post":
        return tuple(ctx.chart_geometry(s["uv"], s["h"])) + tuple(ctx.chart_curvature(s["uv"], s["h"]))
    if s["kind"] == "multiscale":
        return ctx.eval_multiscale(s["x"])
    return ctx.chart_interp(s["uv"], s["data"], s["to"])


# ------------------------------------------------------------------- work
def work(case):
    """Per pair of the sum 40 operations (displacement, two radial functions, dipole and gradient), per target of the
    octree path its pairs within the cut (about 9.2 nodes per sigma^2 of surface where sigma is half a triangle's
    diameter) and 8 operations per coefficient of its local expansion; the far field of the build is left out."""
    kind, mixed = case["kind"], case.get("mixed", False)
    order = 20 if mixed else 26
    per_target = 40.0 * 9.2 * math.pi * CUT[mixed] ** 2 + 8.0 * (order + 1) ** 2
    if kind == "batch":
        mean = (case["nmax"] ** 2 - case["nmin"] ** 2) / (2.0 * math.log(case["nmax"] / case["nmin"]))
        tris = int(12 * case["surfaces"] * mean)
    else:
        tris = 12 * case["n"] ** 2
    skeleton_bytes = tris * (0.5 * 24 + 12 + 8)
    node_bytes = 12 * tris * 48
    if kind in ("eval", "noalloc"):
        t = case["targets"]
        if not case["fmm"]:
            return {"bytes": t * 56 + node_bytes, "flops": 40.0 * t * 12 * tris}
        if case["mesh"] == "sphere":                 # constant sigma 0.05 on the unit sphere
            per_target = 40.0 * 12 * tris * CUT[mixed] ** 2 * 0.0025 / 4.0 + 8.0 * (order + 1) ** 2
        return {"bytes": t * 56 + (skeleton_bytes if case["step"] else node_bytes), "flops": t * per_target}
    if kind == "project":                            # about three evaluations per chart node
        nodes = tris * case["nodes"]
        return {"bytes": nodes * 33 + skeleton_bytes, "flops": 3.0 * nodes * per_target}
    if kind == "batch":
        nodes, t = tris * case["nodes"], case["surfaces"] * case["targets"]
        return {"bytes": nodes * 33 + t * 60 + skeleton_bytes, "flops": (3.0 * nodes + t) * per_target}
    if kind == "post":                               # one gradient and one Hessian pass (87 operations per pair)
        nodes = tris * case["nodes"]
        return {"bytes": nodes * (8 + 80 + 88) + skeleton_bytes, "flops": nodes * per_target * (1.0 + 87.0 / 40.0)}
    if kind == "multiscale":
        return {"bytes": case["targets"] * 64 + skeleton_bytes, "flops": case["targets"] * per_target}
    rows = tris * case["comps"]
    return {"bytes": 8.0 * rows * (case["nodes"] + case["points"]), "flops": 2.0 * rows * case["nodes"] * case["points"]}


# ------------------------------------------------------------------ exact
MOST_PAIRS = 1.2e10                                  # of an exact sum, about ten seconds


def radial(x):
    """S = gamma(3/2, x) x^(-3/2) and T = gamma(5/2, x) x^(-5/2) (with 1.5 S = x T + e^-x)."""
    e = torch.exp(-x)
    small = x.clamp(max=1.0)
    term, series = torch.full_like(x, 1.0 / 2.5), torch.zeros_like(x)
    for k in range(1, 22):                           # e^-x sum_k x^k / ((5/2)(7/2) ... (5/2 + k))
        series = series + term
        term = term * small / (2.5 + k)
    near = e * series
    big = x.clamp(min=1.0)
    root = big.sqrt()
    eb = torch.exp(-big)
    far = (0.75 * math.sqrt(math.pi) * torch.erf(root) - 1.5 * root * eb - big * root * eb) / (big * big * root)
    T = torch.where(x < 1.0, near, far)
    return (x * T + e) / 1.5, T


def node_arrays(verts, tris, rule):
    p = verts[tris.long()]
    e1, e2 = p[:, 1] - p[:, 0], p[:, 2] - p[:, 0]
    y = p[:, None, 0] + rule[None, :, 0, None] * e1[:, None] + rule[None, :, 1, None] * e2[:, None]
    a = rule[None, :, 2, None] * torch.linalg.cross(e1, e2)[:, None]
    return y.reshape(-1, 3), a.reshape(-1, 3)


def exact_field(x, y, a, sigma):
    """Phi and grad Phi by the sum over every node in 64 bits; sigma per node, or per target (a column)."""
    phi, grad = torch.empty(len(x), dtype=torch.float64, device=DEV), torch.empty_like(x)
    per_target = sigma.ndim == 2
    step = max(1, int(3e7) // len(y))
    for i in range(0, len(x), step):
        s = sigma[i:i + step] if per_target else sigma[None]
        d = [x[i:i + step, k, None] - y[None, :, k] for k in range(3)]
        t = (d[0] * d[0] + d[1] * d[1] + d[2] * d[2]) / (2.0 * s * s)
        S, T = radial(t)
        c = 1.0 / (4.0 * math.sqrt(2.0) * math.pi ** 1.5 * s ** 3)
        ad = a[None, :, 0] * d[0] + a[None, :, 1] * d[1] + a[None, :, 2] * d[2]
        phi[i:i + step] = -(c * ad * S).sum(1)
        w, v = c * ad * T / (s * s), c * S
        for k in range(3):
            grad[i:i + step, k] = (w * d[k] - v * a[None, :, k]).sum(1)
    return phi, grad


def pseudonormals(verts, tris):
    """Angle-weighted mean of the unit normals of the triangles at each vertex."""
    t = tris.long()
    p = verts[t]
    nrm = torch.linalg.cross(p[:, 1] - p[:, 0], p[:, 2] - p[:, 0])
    nrm = nrm / nrm.norm(dim=1, keepdim=True)
    total = torch.zeros(len(verts), dtype=torch.float64, device=DEV)
    H = torch.zeros_like(verts)
    for k in range(3):
        u, v = p[:, (k + 1) % 3] - p[:, k], p[:, (k + 2) % 3] - p[:, k]
        ang = torch.atan2(torch.linalg.cross(u, v).norm(dim=1), (u * v).sum(1))
        total.index_add_(0, t[:, k], ang)
        H.index_add_(0, t[:, k], ang[:, None] * nrm)
    return H / total[:, None]


def exact_charts(s, rule):
    """h and x = T + h H with Phi(x) = 1/2 by Newton's method on the exact sum."""
    v, t, uv = s["verts"], s["tris"], s["uv"]
    y, a = node_arrays(v, t, rule)
    sig = s["sigma"].expand(len(t)).repeat_interleave(len(rule))
    b = torch.stack([1.0 - uv.sum(1), uv[:, 0], uv[:, 1]], 1)
    T = (b[None, :, :, None] * v[t.long()][:, None]).sum(2).reshape(-1, 3)
    H = (b[None, :, :, None] * pseudonormals(v, t)[t.long()][:, None]).sum(2).reshape(-1, 3)
    h = torch.zeros(len(T), dtype=torch.float64, device=DEV)
    for _ in range(6):
        phi, grad = exact_field(T + h[:, None] * H, y, a, sig)
        h = h - (phi - 0.5) / (grad * H).sum(1)
    return h, T + h[:, None] * H


def exact(case, seed):
    kind = case["kind"]
    tris = 12 * case.get("n", 0) ** 2
    if kind in ("batch", "post"):
        return None
    if kind == "interp":
        s = inputs(case, seed)

        def basis(uv):                               # products of Legendre polynomials of total degree <= p
            p = round((math.sqrt(8 * case["nodes"] + 1) - 3) / 2)
            uv = uv.cpu().numpy().astype(np.longdouble)
            u = np.polynomial.legendre.legvander(2.0 * uv[:, 0] - 1.0, p)
            v = np.polynomial.legendre.legvander(2.0 * uv[:, 1] - 1.0, p)
            return np.stack([u[:, i] * v[:, j] for j in range(p + 1) for i in range(p + 1 - j)], 1)

        B, E = basis(s["uv"]), basis(s["to"])
        A = np.zeros((case["points"], case["nodes"]), np.longdouble)
        for _ in range(4):                           # A B = E, refined with extended-precision residuals
            A = A + np.linalg.solve(B.T.astype(np.float64), (E - A @ B).T.astype(np.float64)).T
        A = A.astype(np.float64)
        f = s["data"].reshape(tris, case["nodes"], case["comps"])
        out = torch.matmul(f.transpose(1, 2).reshape(-1, case["nodes"]), torch.tensor(A, device=DEV).T.contiguous())
        return out.reshape(tris, case["comps"], case["points"]).transpose(1, 2).reshape(-1, case["comps"]).contiguous()
    count = 7 * tris * case["nodes"] if kind == "project" else case["targets"]
    if float(count) * 12 * tris > MOST_PAIRS:
        return None
    s, rule = inputs(case, seed), torch.tensor(dunavant6(), device=DEV)
    if kind == "project":
        return exact_charts(s, rule) + (None,)
    y, a = node_arrays(s["verts"], s["tris"], rule)
    if kind == "multiscale":
        return exact_multiscale(s, y, a)
    sig = s["sigma"].expand(len(s["tris"])).repeat_interleave(len(rule))
    return exact_field(s["x"], y, a, sig)


def exact_multiscale(s, y, a, lam=2.5):
    """Phi and sigma(x) with the blended width; grad Phi by differentiating through sigma(x) is left out."""
    D = diameters(s["verts"], s["tris"])
    c = s["verts"][s["tris"].long()].mean(1)
    s0 = math.sqrt(5.0) * float(D.max())
    sig = torch.empty(len(s["x"]), dtype=torch.float64, device=DEV)
    step = max(1, int(5e7) // len(c))
    for i in range(0, len(sig), step):
        d2 = (s["x"][i:i + step, None, 0] - c[None, :, 0]).square()
        for k in (1, 2):
            d2 = d2 + (s["x"][i:i + step, None, k] - c[None, :, k]).square()
        w = torch.exp(-(d2 - d2.min(1, keepdim=True).values) / (2.0 * s0 * s0))
        sig[i:i + step] = (w * (D / lam)).sum(1) / w.sum(1)
    return exact_field(s["x"], y, a, sig[:, None])[0], None, sig
