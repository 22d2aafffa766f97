"""The walked tree where its kind changes: every surface split or groups of
them (more than 256 surfaces of fewer than eight triangles), the split's boxes in LDS or in memory, none above 8192 surfaces."""
import numpy as np
import pytest

from paper_2402_13034_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_2402_13034_amd import risrt
    with risrt.Context(0) as c:
        yield c


def _faces(n_surf, per, extra, seed):
    """n_surf rectangles facing the axes, of `per` triangles each (a fan around
    the centre), the last one with `extra` more, in a 12 x 10 x 3 m room."""
    rng = np.random.default_rng(seed)
    V, T, surf = [], [], []
    for s in range(n_surf):
        k = per + (extra if s == n_surf - 1 else 0)
        axis = int(rng.integers(3))
        u, v = (axis + 1) % 3, (axis + 2) % 3
        c = rng.uniform((0.5, 0.5, 0.2), (11.5, 9.5, 2.8))
        h = rng.uniform(0.02, 0.25, 2)
        # k + 2 corners of a convex outline, from one corner
        a = 2 * np.pi * np.arange(k + 2) / (k + 2) + 0.3
        p = np.repeat(c[None], k + 2, 0)
        p[:, u] += h[0] * np.cos(a)
        p[:, v] += h[1] * np.sin(a)
        b = sum(len(x) for x in V)
        V.append(p)
        T.append(b + np.c_[np.zeros(k, int), np.arange(1, k + 1), np.arange(2, k + 2)])
        surf += [s] * k
    V, T = np.concatenate(V).astype(np.float32), np.concatenate(T).astype(np.int32)
    return synth.Scene(V, T, rng.uniform(0.3, 0.8, len(T)).astype(np.float32), np.zeros(len(T), np.float32),
                       np.array(surf, np.int32))


@pytest.mark.parametrize("n_surf,per,extra", [(256, 1, 0), (257, 1, 0), (257, 8, -1), (257, 8, 0), (320, 1, 1),
                                              (321, 2, 1), (2048, 2, 0), (2048, 8, 0), (2049, 2, 0), (4096, 1, 0),
                                              (4097, 1, 0), (2049, 8, -1), (2049, 8, 0), (5000, 8, 1), (8192, 1, 0),
                                              (8192, 8, -1), (8192, 8, 0), (8193, 8, 0)])
def test_equals_brute_force(ctx, n_surf, per, extra):
    from paper_2402_13034_amd import risrt
    p = synth.lab_room(nx=4, ny=3, n_rays=3_000, order=1)
    p.scene = _faces(n_surf, per, extra, n_surf)
    p.ris.elems = p.ris.elems[:7].copy()
    p.gamma = p.gamma[:7].copy()
    print("case trees", n_surf, per, extra, p.scene.n_tri, flush=True)
    outs = []
    for brute in (0, risrt.FLAG_BRUTE_FORCE):
        scene, ris = risrt.upload_problem(ctx, p)
        ch, _ = risrt.trace_problem(ctx, p, scene, ris, flags=risrt.FLAG_KEEP_HITS | risrt.FLAG_KEEP_PATHS | brute)
        E, H = ctx.channel_read(ch)
        outs.append((ctx.hits_read(ch, 0, 1), ctx.hits_read(ch, 1, 1), E, H, ctx.paths_read(ch)["ris_valid"]))
        for h in (ch, scene, ris):
            ctx.destroy(h)
    for a, b in zip(*outs):
        assert np.array_equal(a, b)
    assert (outs[0][0] >= 0).any() and (outs[0][1] >= 0).any()
