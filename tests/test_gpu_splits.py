"""The splits of the evaluation kernels at the sizes where a wrong range would
show: one target, partly filled waves and tiles, node counts that leave a
remainder of a chunk, ragged batches, and the counts on both sides of the rule
that chooses a split."""
import numpy as np
import pytest

import oracle
import paper_1909_13356_amd as lss
from workloads import dunavant6, cube_mesh, star_surface, triangle_diameters, bbox_targets, chart_nodes, configs

pytestmark = pytest.mark.gpu


def _err(a, b):
    return np.abs(a - b).max() / np.abs(b).max()


# bars of the two precisions against the oracle (relative to the largest value)
BAR = {lss.FP64: 1e-12, lss.MIXED: 1e-6}


@pytest.mark.parametrize("prec", [lss.FP64, lss.MIXED])
@pytest.mark.parametrize("n", [1, 64, 257, 4099])
def test_direct_split_against_oracle(n, prec):
    v, t = cube_mesh(9)                              # 972 triangles, 11 664 nodes: 45.6 chunks of 256
    x = bbox_targets(v, n, pad=0.5, seed=n)
    rule = dunavant6()
    c = lss.Context()
    c.set_options(precision=prec)
    c.set_sources(v, t, rule)
    c.set_sigma(0.1)
    phi, grad = c.eval(x)
    k = np.linspace(0, n - 1, min(n, 200)).astype(int)
    # relative to the sum of the terms' magnitudes: one far target's Phi is all cancellation
    op, og, ap, ag = oracle.evaluate(v, t, np.full(len(t), 0.1), rule, x[k], with_abs=True)
    assert (np.abs(phi[k] - op) <= BAR[prec] * ap).all() and (np.abs(grad[k] - og).max(1) <= BAR[prec] * ag).all()
    assert c.stats()["last_pairs"] == n * 12 * len(t)
    phi2, _ = c.eval(x, want_grad=False)
    assert np.array_equal(phi, phi2)


@pytest.mark.parametrize("prec", [lss.FP64, lss.MIXED])
def test_direct_split_matches_unsplit(prec):
    """The same targets among 170 000 (one workgroup per tile: no split) and alone; a tile's origin and a partial
    sum's chunk move, so the results agree to the rounding of the sums (1e-13 FP64, 1e-6 mixed: the bar)."""
    parts = [star_surface(5, seed=1), star_surface(3, seed=2)]
    meshes = [dict(verts=v, tris=t, sigma=0.5 * triangle_diameters(v, t),
                   targets=bbox_targets(v, m, seed=7 + m)) for (v, t), m in zip(parts, (169_000, 1_000))]
    b = configs.concat_batch(meshes)
    c = lss.Context()
    c.set_options(precision=prec)
    c.set_sources(b["verts"], b["tris"], dunavant6(), tri_offsets=b["tri_offsets"])
    c.set_sigma(b["sigma"])
    p0, g0 = c.eval(b["targets"], x_mesh=b["target_mesh"])
    k = np.concatenate([np.arange(0, 169_000, 400), np.arange(169_000, 170_000, 3)])
    p1, g1 = c.eval(b["targets"][k], x_mesh=b["target_mesh"][k])
    tol = {lss.FP64: 1e-13, lss.MIXED: 1e-6}[prec]
    assert _err(p1, p0[k]) <= tol and _err(g1, g0[k]) <= tol


def _forest(flip=lambda x: x):
    """Two star surfaces and a cube too small for any translation, their coordinates mapped by `flip`."""
    parts = [(star_surface(14, seed=5), 4000), (star_surface(9, seed=6), 1500), (cube_mesh(1), 100)]
    return configs.concat_batch([dict(verts=flip(v), tris=t, sigma=0.12 * triangle_diameters(v, t),
                                      targets=flip(bbox_targets(v, m, seed=m))) for (v, t), m in parts])


@pytest.mark.parametrize("p,K", [(26, 7), (26, 18), (40, 8)])
def test_m2l_against_direct(p, K):
    """At orders whose truncation is below rounding the field of a ragged forest equals the exact sum (1e-12), and a
    rebuild, which reuses the plan's buffers and operators, gives the same bits."""
    b = _forest()
    c = lss.Context()
    c.set_sources(b["verts"], b["tris"], dunavant6(), tri_offsets=b["tri_offsets"])
    c.set_sigma(b["sigma"])
    p0, g0 = c.eval(b["targets"], x_mesh=b["target_mesh"])
    c.set_options(far_field=lss.FAR_FMM, fmm_order=p, admissibility=K)
    p1, g1 = c.eval(b["targets"], x_mesh=b["target_mesh"])
    assert c.stats()["n_m2l"] > 1000
    assert _err(p1, p0) <= 1e-12 and _err(g1, g0) <= 1e-12
    c.set_sigma(b["sigma"])
    p2, g2 = c.eval(b["targets"], x_mesh=b["target_mesh"])
    assert np.array_equal(p1, p2) and np.array_equal(g1, g2)


@pytest.mark.parametrize("p", [2, 3, 7, 11, 20, 26])
def test_m2l_symmetry(p):
    """A quarter turn about z and a reflection z -> -z map the octree onto itself and every displacement to another of
    its group, and the series truncated at order p onto the truncated series: the field at the mapped targets is the
    mapped field to rounding (1e-12 of the largest value, orders around the tile and padding sizes)."""
    got = []
    for turn in (lambda x: x, lambda x: np.stack([-x[:, 1], x[:, 0], -x[:, 2]], 1)):
        b = _forest(turn)
        b["tris"] = b["tris"] if not got else np.ascontiguousarray(b["tris"][:, ::-1])   # a reflection turns them over
        c = lss.Context()
        c.set_options(far_field=lss.FAR_FMM, fmm_order=p, leaf_capacity=32)
        c.set_sources(b["verts"], b["tris"], dunavant6(), tri_offsets=b["tri_offsets"])
        c.set_sigma(b["sigma"])
        got.append(c.eval(b["targets"], x_mesh=b["target_mesh"]))
    (p0, g0), (p1, g1) = got
    assert _err(p1, p0) <= 1e-12
    assert _err(np.stack([g1[:, 1], -g1[:, 0], -g1[:, 2]], 1), g0) <= 1e-12


@pytest.mark.parametrize("prec", [lss.FP64, lss.MIXED])
@pytest.mark.parametrize("n", [1, 65, 3000, 150_000])
def test_fmm_tiles_shared_by_waves(n, prec):
    """The octree evaluation with few tiles (every tile heavy: a workgroup each), and with enough that light tiles go to
    single waves, on a ragged pair of surfaces with targets inside and outside the root cubes: the exact sum to the
    precision's bar, and the same bits on a second call."""
    parts = [star_surface(13, seed=3), star_surface(6, seed=4)]
    meshes = [dict(verts=v, tris=t, sigma=0.5 * triangle_diameters(v, t),
                   targets=bbox_targets(v, m, pad=p, seed=m)) for (v, t), m, p in zip(parts, (n, n // 3 + 1), (0.1, 3.0))]
    b = configs.concat_batch(meshes)
    c = lss.Context()
    c.set_sources(b["verts"], b["tris"], dunavant6(), tri_offsets=b["tri_offsets"])
    c.set_sigma(b["sigma"])
    c.set_options(precision=prec, far_field=lss.FAR_FMM)
    x, xm = b["targets"], b["target_mesh"]
    p1, g1 = c.eval(x, x_mesh=xm)
    p2, g2 = c.eval(x, x_mesh=xm)
    assert np.array_equal(p1, p2) and np.array_equal(g1, g2)
    k = np.unique(np.linspace(0, len(x) - 1, 3000).astype(int))
    c.set_options(precision=lss.FP64)
    p0, g0 = c.eval(x[k], x_mesh=xm[k])
    # |Phi| <= 1 inside and the gradient reaches 1 / (sqrt(2 pi) sigma) at the surface: the natural scales, also for
    # few targets far from it
    scale = 1.0 / (np.sqrt(2.0 * np.pi) * b["sigma"].max())
    assert np.abs(p1[k] - p0).max() <= BAR[prec] and np.abs(g1[k] - g0).max() <= BAR[prec] * scale


@pytest.mark.parametrize("n", [1, 63, 2500, 60_000])
def test_hessian_and_multiscale_tiles_shared_by_waves(n):
    """The Hessian and the target-attached width through the octree against their every-pair paths, for few targets (a
    workgroup per tile) and many (light tiles by single waves).  Bars: 1e-11 of the natural scale for the Hessian (its
    cut truncates the third radial function at 2e-11 relative), 1e-12 for Phi, grad Phi and the multiscale field."""
    v, t = star_surface(12, seed=8)
    x = bbox_targets(v, n, pad=0.3, seed=n)
    sig = 0.5 * triangle_diameters(v, t)
    scale = 1.0 / (np.sqrt(2.0 * np.pi) * sig.min())
    got = []
    for far in (lss.FAR_DIRECT, lss.FAR_FMM):
        c = lss.Context()
        c.set_options(far_field=far)
        c.set_sources(v, t, dunavant6())
        c.set_sigma(sig)
        got.append(c.eval_hessian(x) + c.eval_multiscale(x, 2.5, 0.1))
    for k, (a, b, tol) in enumerate(zip(got[1], got[0], (1e-12, 1e-12 * scale, 1e-11 * scale / sig.min(),
                                                         1e-12, 1e-12 * scale, 1e-12))):
        assert np.abs(a - b).max() <= tol, k


def test_mixed_heavy_tiles_are_the_same_bits():
    """Tiles taken by a whole workgroup (few targets) and by single waves (the same targets beside many of another mesh
    of the batch, which make them light) give the same bits: the mixed projection depends on it."""
    parts = [star_surface(13, seed=3), star_surface(12, seed=4)]
    sig = [0.5 * triangle_diameters(v, t) for v, t in parts]
    few = bbox_targets(parts[0][0], 5000, pad=0.1, seed=1)
    many = bbox_targets(parts[1][0], 1_500_000, pad=0.02, seed=2)
    b = configs.concat_batch([dict(verts=v, tris=t, sigma=s, targets=x)
                              for (v, t), s, x in zip(parts, sig, (few, many))])
    c = lss.Context()
    c.set_sources(b["verts"], b["tris"], dunavant6(), tri_offsets=b["tri_offsets"])
    c.set_sigma(b["sigma"])
    c.set_options(precision=lss.MIXED, far_field=lss.FAR_FMM)
    p0, g0 = c.eval(few, x_mesh=np.zeros(len(few), np.int32))
    p1, g1 = c.eval(b["targets"], x_mesh=b["target_mesh"])
    assert np.array_equal(p0, p1[:len(few)]) and np.array_equal(g0, g1[:len(few)])


@pytest.mark.parametrize("n", [1, 255, 4000, 600_000])
def test_sigma_field_pieces(n):
    """sigma(x) by the direct sum, its centroid runs split over workgroups (few points) and not (6e5), on a ragged pair
    of meshes with runs that straddle them, against the oracle on a sample (1e-12 relative)."""
    parts = [star_surface(9, seed=1), star_surface(5, seed=2)]
    meshes = [dict(verts=v, tris=t, sigma=0.5 * triangle_diameters(v, t), targets=bbox_targets(v, m, pad=0.5, seed=m))
              for (v, t), m in zip(parts, (n, n // 2 + 1))]
    b = configs.concat_batch(meshes)
    c = lss.Context()
    c.set_options(far_field=lss.FAR_FMM, sigma_interp=1)
    c.set_sources(b["verts"], b["tris"], dunavant6(), tri_offsets=b["tri_offsets"])
    sig = c.eval_multiscale(b["targets"], 2.5, 0.07, x_mesh=b["target_mesh"])[2]
    k = np.unique(np.linspace(0, len(sig) - 1, 300).astype(int))
    want = oracle.sigma_field(b["verts"], b["tris"], b["targets"][k], 2.5, 0.07, tri_offsets=b["tri_offsets"],
                              x_mesh=b["target_mesh"][k])
    want = want[0] if isinstance(want, tuple) else want
    assert np.abs(sig[k] / want - 1.0).max() <= 1e-12


@pytest.mark.parametrize("p,ne,ncomp,n,bad", [(0, 1, 1, 2, False), (1, 16, 3, 4, False), (4, 17, 2, 5, True), (8, 66, 3, 7, True),
                                              (8, 81, 16, 3, False), (5, 700, 5, 3, True), (19, 33, 1, 3, False),
                                              (19, 200, 10, 2, True), (19, 9, 15, 2, False), (8, 66, 3, 40, False), (9, 20, 3, 4, True), (14, 33, 1, 3, False),
                                              (15, 33, 1, 3, False)])
def test_chart_interp_tiles(p, ne, ncomp, n, bad):
    """Chart interpolation at the edges of the matrix tiles: one point and one node, a full tile, remainders in points,
    nodes and columns, points shared by workgroups, the matrix from memory, a triangle too large for LDS.  A node that
    is not finite stays with its own triangle and component.  Bound: both solve with V, so 64 ulp
    times its condition number, relative to the sums of magnitudes."""
    v, t = star_surface(n, seed=n)
    c = lss.Context()
    c.set_sources(v, t, dunavant6())
    uv = chart_nodes(p) if p else np.array([[0.3, 0.3]])
    rng = np.random.default_rng(ne)
    ev = rng.dirichlet([1, 1, 1], ne)[:, :2]
    f = rng.standard_normal((len(t) * len(uv), ncomp))
    if bad:
        f[len(uv) // 2, ncomp - 1], f[-1, 0] = np.nan, np.inf
    got = c.chart_interp(uv, f, ev)
    I = oracle.chart_interp(uv, np.eye(len(uv)).reshape(-1), ev).reshape(len(uv), ne).T      # one triangle per node
    ff = f.reshape(len(t), len(uv), ncomp)
    want = np.einsum("ei,jic->jec", I, np.where(np.isfinite(ff), ff, 0.0))
    scale = np.einsum("ei,jic->jec", np.abs(I), np.where(np.isfinite(ff), np.abs(ff), 0.0)).max()
    hit = ~np.isfinite(ff).all(axis=1)                                                       # (triangle, component)
    got = got.reshape(len(t), ne, ncomp)
    mask = np.broadcast_to(hit[:, None, :], got.shape)
    assert np.all(np.isfinite(got[~mask])) and not np.any(np.isfinite(got[mask]))
    assert np.abs(got - want)[~mask].max() <= 64 * 2.0 ** -52 * np.linalg.cond(oracle.koornwinder(uv, p)) * scale


@pytest.mark.parametrize("n", [2, 17])
def test_m2l_forms_alternate(n):
    """A mixed context's field (M2L by class) before and after a target-attached evaluation (one plan of all pairs, also
    where there is no pair at all): the same bit for bit, and the latter against the direct sum (1e-7, its cut)."""
    v, t = star_surface(n, seed=n)
    x = bbox_targets(v, 800, pad=0.2, seed=3)
    c = lss.Context()
    c.set_options(precision=lss.MIXED, far_field=lss.FAR_FMM)
    c.set_sources(v, t, dunavant6())
    c.set_sigma(0.5 * triangle_diameters(v, t))
    before = c.eval(x)
    ms = c.eval_multiscale(x, 2.5, 0.0)
    after = c.eval(x)
    assert all(np.array_equal(a, b) for a, b in zip(before, after))
    want = oracle.evaluate_multiscale(v, t, dunavant6(), x, 2.5, 0.0)
    assert np.abs(ms[0] - want[0]).max() <= 1e-7


@pytest.mark.parametrize("precision,order", [(lss.FP64, 26), (lss.FP64, 9), (lss.MIXED, 20), (lss.MIXED, 6)])
def test_translation_launch_sizes(precision, order):
    """The far field of one small surface (short translation launches, contraction lengths that end inside a step) and
    of 40 copies of it in one context (long ones): the products are the same, summed in the same order but for the
    classes that change their form with the number of pairs (1e-13 of the largest value)."""
    v, t = star_surface(10, seed=6)
    sig = 0.5 * triangle_diameters(v, t)
    x = bbox_targets(v, 500, pad=0.1, seed=2)
    one = dict(verts=v, tris=t, sigma=sig, targets=x)
    b = configs.concat_batch([one] * 40)
    out = []
    for m in (one, b):
        c = lss.Context()
        c.set_options(precision=precision, far_field=lss.FAR_FMM, fmm_order=order)
        kw = {} if m is one else dict(tri_offsets=b["tri_offsets"])
        c.set_sources(m["verts"], m["tris"], dunavant6(), **kw)
        c.set_sigma(m["sigma"])
        out.append(c.eval(m["targets"], **({} if m is one else dict(x_mesh=b["target_mesh"]))))
    for a, w in zip(out[0], out[1]):
        w = w.reshape((40,) + a.shape)
        assert np.abs(w - a[None]).max() <= 1e-13 * np.abs(a).max()


@pytest.mark.parametrize("precision,order", [(lss.FP64, 1), (lss.FP64, 2), (lss.FP64, 3), (lss.FP64, 17), (lss.FP64, 40),
                                             (lss.MIXED, 17), (lss.MIXED, 40)])
def test_expansion_orders(precision, order):
    """Expansions evaluated by a wave, from the lowest order (columns of one and two terms) to the highest: the field of
    the tile loop against that of the fixed tiles (FP64: tile=128, another kernel with the same expansions, 1e-13 of the
    largest value), and mixed against FP64 at the same order, admissibility, leaf size and cut (2e-6)."""
    v, t = star_surface(12, seed=9)
    x = bbox_targets(v, 700, pad=0.1, seed=4)
    out = []
    for kw in (dict(precision=lss.FP64, tile=128),
               dict(precision=precision, tile=0) if precision == lss.FP64 else
               dict(precision=precision, admissibility=7, leaf_shrink=2.0)):
        c = lss.Context()
        c.set_options(far_field=lss.FAR_FMM, fmm_order=order, **kw)
        c.set_sources(v, t, dunavant6())
        c.set_sigma(0.5 * triangle_diameters(v, t))
        out.append(c.eval(x))
    tol = 1e-13 if precision == lss.FP64 else 2e-6
    for a, b in zip(*out):
        assert np.abs(a - b).max() <= tol * np.abs(a).max()


def test_m2l_products_are_bounded():
    """A volume's triangles beside 4000 meshes whose boxes have no pair: the M2L products of one launch stay within 2 GiB
    however the pairs are spread over the boxes (the build takes less than 4 GiB in all; 1.4 GiB are expansions, lists
    and records), and the field equals the direct sum (1e-12)."""
    torch = pytest.importorskip("torch")
    rng = np.random.default_rng(3)
    m = 18_000
    v = (rng.random((m, 1, 3)) + 0.01 * rng.standard_normal((m, 3, 3))).reshape(-1, 3)
    t = np.arange(3 * m, dtype=np.int32).reshape(m, 3)
    cube = cube_mesh(1)
    small = dict(verts=cube[0], tris=cube[1], sigma=np.full(len(cube[1]), 1e-3), targets=np.zeros((0, 3)))
    b = configs.concat_batch([dict(verts=v, tris=t, sigma=np.full(m, 1e-3), targets=rng.random((500, 3)))] + [small] * 4000)
    free = torch.cuda.mem_get_info()[0]
    c = lss.Context()
    c.set_options(far_field=lss.FAR_FMM, leaf_capacity=100)
    c.set_sources(b["verts"], b["tris"], dunavant6(), tri_offsets=b["tri_offsets"])
    c.set_sigma(b["sigma"])
    c.build()
    assert free - torch.cuda.mem_get_info()[0] < 4 << 30
    assert c.stats()["n_m2l"] > 1_000_000
    got = c.eval(b["targets"], x_mesh=b["target_mesh"])
    c.set_options(far_field=lss.FAR_DIRECT)
    want = c.eval(b["targets"], x_mesh=b["target_mesh"])
    assert _err(got[0], want[0]) <= 1e-12 and _err(got[1], want[1]) <= 1e-12


def test_multiscale_is_the_same_in_both_precisions():
    """The target-attached width is summed in FP64 in either precision: with the same tree the same bits.  At 60 000
    targets some tiles are shared by a workgroup's waves, which add their totals, and most are not; which ones must not
    depend on the context's precision."""
    v, t = star_surface(24, seed=8)
    x = bbox_targets(v, 60_000, pad=0.1, seed=5)
    out = []
    for prec in (lss.FP64, lss.MIXED):
        c = lss.Context()
        c.set_options(precision=prec, far_field=lss.FAR_FMM, fmm_order=18, cut_factor=7.0, leaf_capacity=64,
                      leaf_shrink=2.0, admissibility=5, sigma_interp=1)
        c.set_sources(v, t, dunavant6())
        out.append(c.eval_multiscale(x, 2.5, 0.0))
    assert all(np.array_equal(a, b) for a, b in zip(*out))


def test_chart_interp_gives_a_large_matrix_back():
    """The matrix to 2^20 points (0.4 GB) is not held by the context after the call: less than 128 MiB stay (64 MiB at
    most of it), and the values are those of a call with few of the points (1e-12)."""
    torch = pytest.importorskip("torch")
    v, t = cube_mesh(1)
    uv, rng = chart_nodes(8), np.random.default_rng(4)
    ev = rng.dirichlet([1, 1, 1], 1 << 20)[:, :2]
    f = rng.standard_normal(len(t) * len(uv))
    c = lss.Context()
    c.set_sources(v, t, dunavant6())
    few = c.chart_interp(uv, f, ev[:: 1 << 10]).reshape(len(t), -1)
    free = torch.cuda.mem_get_info()[0]
    got = c.chart_interp(uv, f, ev).reshape(len(t), -1)
    assert free - torch.cuda.mem_get_info()[0] < 128 << 20
    assert np.abs(got[:, :: 1 << 10] - few).max() <= 1e-12 * np.abs(few).max()


def test_sigma_field_pieces_of_several_runs():
    """1e5 points and 76 runs of 256 centroids, split in five: pieces of several runs, a short last one, and in the
    second mesh (eleven runs, the first shared with the other mesh) one without any.  A point's nearest centroid lies in
    one of them, so the merge rescales the others.  Against the oracle on a sample (1e-12 relative)."""
    parts = [star_surface(29, seed=1), star_surface(11, seed=2)]
    meshes = [dict(verts=v, tris=t, sigma=0.5 * triangle_diameters(v, t), targets=bbox_targets(v, m, pad=0.5, seed=m))
              for (v, t), m in zip(parts, (66_000, 33_001))]
    b = configs.concat_batch(meshes)
    c = lss.Context()
    c.set_options(far_field=lss.FAR_FMM, sigma_interp=1)
    c.set_sources(b["verts"], b["tris"], dunavant6(), tri_offsets=b["tri_offsets"])
    sig = c.eval_multiscale(b["targets"], 2.5, 0.07, x_mesh=b["target_mesh"])[2]
    k = np.unique(np.linspace(0, len(sig) - 1, 300).astype(int))
    want = oracle.sigma_field(b["verts"], b["tris"], b["targets"][k], 2.5, 0.07, tri_offsets=b["tri_offsets"],
                              x_mesh=b["target_mesh"][k])
    want = want[0] if isinstance(want, tuple) else want
    assert np.abs(sig[k] / want - 1.0).max() <= 1e-12


@pytest.mark.parametrize("prec", [lss.FP64, lss.MIXED])
def test_direct_workspace_holds_for_fewer_targets(prec):
    """A direct sum's workspace is allocated once: calls of fewer targets, some of which have more targets times pieces
    (104 000 in 5 against 110 000 in 4), take no more memory."""
    torch = pytest.importorskip("torch")
    v, t = cube_mesh(9)
    x = torch.as_tensor(bbox_targets(v, 110_000, pad=0.5, seed=3), device="cuda")
    phi, grad = torch.empty_like(x[:, 0].contiguous()), torch.empty_like(x)
    c = lss.Context()
    c.set_options(precision=prec)
    c.set_sources(v, t, dunavant6())
    c.set_sigma(0.1)
    c.eval(x, phi=phi, grad=grad)
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    for n in (104_000, 80_000, 4096, 1):
        c.eval(x[:n], phi=phi[:n], grad=grad[:n])
        torch.cuda.synchronize()
        assert torch.cuda.mem_get_info()[0] == free, n


@pytest.mark.parametrize("n,seed", [(12, 1), (20, 1), (20, 3)])
def test_expansion_sums_round_no_more_than_term_by_term(n, seed):
    """FP64: the rms error of Phi against the direct sum with the expansions of the tile loop (products fused into a sum
    per column) is no larger than with those of the 128-target tiles (one rounding per term).  The rest of the error is
    the same; 0.5% for the order of the near sums."""
    v, t = star_surface(n, seed=seed)
    x = bbox_targets(v, 40_000, pad=0.05, seed=seed)
    out = []
    for kw in (dict(far_field=lss.FAR_DIRECT), dict(far_field=lss.FAR_FMM, tile=0), dict(far_field=lss.FAR_FMM, tile=128)):
        c = lss.Context()
        c.set_options(**kw)
        c.set_sources(v, t, dunavant6())
        c.set_sigma(0.5 * triangle_diameters(v, t))
        out.append(c.eval(x)[0])
    wave, fixed = (np.sqrt(((p - out[0]) ** 2).mean()) for p in out[1:])
    assert wave <= 1.005 * fixed
