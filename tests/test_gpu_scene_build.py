"""The scene build at the edges of its tiles: the node boxes (one workgroup per
2048 leaves, the nodes above by leaf range), the tree above the surfaces (one
workgroup, then one per 256 surfaces; boxes in LDS up to 2048; none above 8192)
and the surface tables (lanes over a surface's triangles) give the walk that
testing every triangle gives."""
import numpy as np
import pytest

from paper_2402_13034_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_2402_13034_amd import risrt
    with risrt.Context(0) as c:
        yield c


def _trimmed(n_tri, sub):
    """The lab room cut at n_tri triangles (whole surfaces renumbered)."""
    p = synth.lab_room(nx=4, ny=4, sub=sub, n_rays=20_000, order=2)
    sc = p.scene
    assert sc.n_tri >= n_tri
    surf = np.unique(sc.surf[:n_tri], return_inverse=True)[1].astype(np.int32)
    p.scene = synth.Scene(sc.V, sc.T[:n_tri].copy(), sc.refl_re[:n_tri].copy(), sc.refl_im[:n_tri].copy(), surf)
    return p


# one tile less a leaf, a full one, one leaf and some leaves into the next, a third tile of one leaf; surfaces of
# 18, 72 and 162 triangles (below, above and over twice a wave)
@pytest.mark.parametrize("n_tri,sub", [(2, 3), (1908, 3), (2047, 6), (2048, 6), (2049, 6), (4097, 6), (5000, 9),
                                       (17000, 9)])
def test_build_equals_brute_force(ctx, n_tri, sub):
    from paper_2402_13034_amd import risrt
    prob = _trimmed(n_tri, sub)
    print("case build", n_tri, sub, flush=True)
    outs = []
    for brute in (0, risrt.FLAG_BRUTE_FORCE):
        scene, ris = risrt.upload_problem(ctx, prob)
        ch, _ = risrt.trace_problem(ctx, prob, scene, ris,
                                    flags=risrt.FLAG_KEEP_HITS | risrt.FLAG_KEEP_PATHS | brute)
        E, H = ctx.channel_read(ch)
        p = ctx.paths_read(ch)
        outs.append((ctx.hits_read(ch, 0, 2), ctx.hits_read(ch, 1, 2), E, H, p["env"], p["ris_valid"]))
        for h in (ch, scene, ris):
            ctx.destroy(h)
    for a, b in zip(*outs):
        assert np.array_equal(a, b)
    # the reflection triangle of every path: the grid lists against the oracle's scan of the whole surface
    from oracle import oracle as O
    with O.accelerated():
        ref = O.trace(prob)
    assert np.array_equal(outs[0][4]["tri"][:, :2], ref["env_tri"][:, :2])
    assert np.array_equal(outs[0][5], ref["ris_valid"])


# every triangle a surface of its own: the surface counts at which the tree above them changes its way
@pytest.mark.parametrize("n_surf", [2, 3, 256, 257, 2048, 2049, 8192, 8193])
def test_tree_above_surfaces(ctx, n_surf):
    from paper_2402_13034_amd import risrt
    p = _trimmed(n_surf, 7)
    p.order = 1
    p.n_rays = 4_000
    p.scene.surf = np.arange(n_surf, dtype=np.int32)
    print("case surfaces", n_surf, flush=True)
    outs = []
    for brute in (0, risrt.FLAG_BRUTE_FORCE):
        scene, ris = risrt.upload_problem(ctx, p)
        ch, st = risrt.trace_problem(ctx, p, scene, ris, flags=risrt.FLAG_KEEP_HITS | risrt.FLAG_KEEP_PATHS | brute)
        E, H = ctx.channel_read(ch)
        outs.append((ctx.hits_read(ch, 0, 1), ctx.hits_read(ch, 1, 1), E, H, ctx.paths_read(ch)["ris_valid"]))
        for h in (ch, scene, ris):
            ctx.destroy(h)
    for a, b in zip(*outs):
        assert np.array_equal(a, b)


# either side of the line between four lanes per ray and a wave per 64 rays, at orders of one- and two-word keys
@pytest.mark.parametrize("n_tri,n_rays,order", [(63, 3_000, 2), (64, 3_000, 2), (1908, 50_000, 3), (1908, 90_000, 3),
                                                (1908, 20_000, 5), (1, 500, 1)])
def test_discovery_lanes_per_ray(ctx, n_tri, n_rays, order):
    from paper_2402_13034_amd import risrt
    p = _trimmed(max(n_tri, 2), 3)
    if n_tri == 1:
        p.scene = synth.Scene(p.scene.V, p.scene.T[:1].copy(), p.scene.refl_re[:1].copy(), p.scene.refl_im[:1].copy(),
                              np.zeros(1, np.int32))
    p.order, p.n_rays = order, n_rays
    print("case discovery", n_tri, n_rays, order, flush=True)
    outs = []
    for brute in (0, risrt.FLAG_BRUTE_FORCE):
        scene, ris = risrt.upload_problem(ctx, p)
        ch, st = risrt.trace_problem(ctx, p, scene, ris, flags=risrt.FLAG_KEEP_HITS | brute)
        outs.append((ctx.hits_read(ch, 0, order), ctx.hits_read(ch, 1, order), ctx.candidates_read(ch, 0),
                     ctx.candidates_read(ch, 1), st["discovery_segments"], *ctx.channel_read(ch)))
        for h in (ch, scene, ris):
            ctx.destroy(h)
    for a, b in zip(*outs):
        assert np.array_equal(a, b)


def test_counting_walk_is_the_morton_tree(ctx):
    """The counting builds walk the scene's Morton tree, whose boxes are made
    for them: the same hits and fields, and work that does not change between
    a scene and the same one rebuilt."""
    from paper_2402_13034_amd import risrt
    p = _trimmed(5000, 6)
    got = []
    for flags in (0, risrt.FLAG_COUNT_WORK, risrt.FLAG_COUNT_WORK):
        scene, ris = risrt.upload_problem(ctx, p)
        ch, st = risrt.trace_problem(ctx, p, scene, ris, flags=flags)
        got.append((ctx.channel_read(ch), st["ris_work"] + st["discovery_work"], st["leg_segments"]))
        for h in (ch, scene, ris):
            ctx.destroy(h)
    for g in got[1:]:
        assert np.array_equal(g[0][0], got[0][0][0]) and np.array_equal(g[0][1], got[0][0][1])
        assert g[2] == got[0][2]
    assert got[1][1] == got[2][1] and min(got[1][1]) > 0


# triangles per face at which the containment grid gets finer (16, 64, 256 cells; 1024 are the most), and a fan whose
# long triangles overlap so many cells that the grid is halved until its lists fit
@pytest.mark.parametrize("mesh,n", [("cells", 2), ("cells", 18), ("cells", 128), ("cells", 242), ("cells", 512),
                                    ("cells", 1152), ("fan", 15), ("fan", 65), ("fan", 300), ("fan", 1500)])
def test_containment_grid(ctx, mesh, n):
    """A box whose faces are single surfaces of n triangles, each with its own
    coefficient: the triangle of every reflection against the oracle's scan of
    the whole surface, fields against the build that scans too."""
    from oracle import oracle as O
    from paper_2402_13034_amd import risrt
    rng = np.random.default_rng(n)
    size = np.array([4.0, 3.0, 2.5])
    V, T, surf = [], [], []
    for axis in range(3):
        for side in (0.0, 1.0):
            o, eu, ev = np.zeros(3), np.zeros(3), np.zeros(3)
            o[axis] = side * size[axis]
            eu[(axis + 1) % 3] = size[(axis + 1) % 3]
            ev[(axis + 2) % 3] = size[(axis + 2) % 3]
            base = sum(len(v) for v in V)
            if mesh == "cells":
                g = int(np.sqrt(n // 2))
                a, b = np.meshgrid(np.arange(g + 1) / g, np.arange(g + 1) / g, indexing="ij")
                i, j = (x.ravel() for x in np.meshgrid(np.arange(g), np.arange(g), indexing="ij"))
                q = i * (g + 1) + j
                tri = np.r_[np.c_[q, q + g + 1, q + 1], np.c_[q + 1, q + g + 1, q + g + 2]]
                pts = np.c_[a.ravel(), b.ravel()]
            else:   # from one corner over the two far edges
                h = n // 2
                e = np.r_[np.c_[np.ones(h), np.arange(h) / h], np.c_[1 - np.arange(n - h) / (n - h), np.ones(n - h)],
                          [[0.0, 1.0]]]
                pts = np.r_[[[0.0, 0.0]], e]
                tri = np.c_[np.zeros(n, int), np.arange(1, n + 1), np.arange(2, n + 2)]
            V.append(o + pts[:, :1] * eu + pts[:, 1:] * ev)
            T.append(base + rng.permutation(tri))
            surf += [2 * axis + int(side)] * len(tri)
    V, T = np.concatenate(V).astype(np.float32), np.concatenate(T).astype(np.int32)
    re = rng.uniform(0.2, 0.9, len(T)).astype(np.float32)
    p = synth.lab_room(nx=3, ny=3, n_rays=4_000, order=2)
    p.scene = synth.Scene(V, T, re, np.zeros_like(re), np.array(surf, np.int32))
    p.tx_pos = np.array([0.7, 0.6, 1.9])
    p.ris.centre = np.array([3.99, 1.5, 1.2])
    p.ris.elems = p.ris.centre + rng.uniform(-0.3, 0.3, (70, 3)) * [0.0, 1.0, 1.0]
    p.gamma = np.ones((70, 1), np.complex128)
    p.rx_pos = rng.uniform(0.1, 0.9, (9, 3)) * size
    print("case grid", mesh, n, flush=True)
    out = []
    for flags in (risrt.FLAG_KEEP_PATHS, risrt.FLAG_COUNT_WORK):
        scene, ris = risrt.upload_problem(ctx, p)
        ch, _ = risrt.trace_problem(ctx, p, scene, ris, flags=flags)
        out.append(ctx.channel_read(ch))
        if flags == risrt.FLAG_KEEP_PATHS:
            kept = ctx.paths_read(ch)
        for h in (ch, scene, ris):
            ctx.destroy(h)
    assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1])
    with O.accelerated():
        ref = O.trace(p)
    assert np.array_equal(kept["env"]["tri"][:, :2], ref["env_tri"][:, :2])
    assert np.array_equal(kept["ris_valid"], ref["ris_valid"])
