"""Deep trees under the walks themselves: the linear BVH of a scene of more than
8192 surfaces with a chain of nested, overlapping groups of triangles (both
children of a level hit, so entries wait at every level of the stacks), a
surface whose own subtree is deeper than 31 levels, and a scene whose tree with
the split above the surfaces is deeper than 63 while its linear BVH is not (the
build then takes the linear BVH)."""
import numpy as np
import pytest

from paper_2402_13034_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_2402_13034_amd import risrt
    with risrt.Context(0) as c:
        yield c


def _scene(V, T, surf, seed):
    V, T, surf = np.concatenate(V).astype(np.float32), np.concatenate(T).astype(np.int32), np.concatenate(surf)
    re = np.random.default_rng(seed).uniform(0.3, 0.8, len(T)).astype(np.float32)
    return synth.Scene(V, T, re, np.zeros_like(re), np.unique(surf, return_inverse=True)[1].astype(np.int32))


def _equals_brute_force(ctx, p, depth, rays):
    from paper_2402_13034_amd import risrt
    for n_rays in rays:
        p.n_rays = n_rays
        outs = []
        for brute in (0, risrt.FLAG_BRUTE_FORCE):
            scene, ris = risrt.upload_problem(ctx, p)
            info = ctx.scene_info(scene)
            assert depth[0] <= info["bvh_depth"] <= depth[1], info
            ch, _ = risrt.trace_problem(ctx, p, scene, ris, flags=risrt.FLAG_KEEP_HITS | risrt.FLAG_KEEP_PATHS | brute)
            E, H = ctx.channel_read(ch)
            k = ctx.paths_read(ch)
            outs.append((ctx.hits_read(ch, 0, p.order), ctx.hits_read(ch, 1, p.order), E, H, k["env"], k["ris_valid"]))
            for h in (ch, scene, ris):
                ctx.destroy(h)
        for a, b in zip(*outs):
            assert np.array_equal(a, b)


def _problem(scene, corner):
    """Rays from a point near the corner, receivers towards it and in the room."""
    p = synth.lab_room(nx=3, ny=2, order=2)
    p.scene = scene
    p.tx_pos = np.array([0.031, 0.027, 0.022])
    p.tx_ant = p.rx_ant
    near = np.array([[0.5, 0.4, 0.3], [0.1, 0.1, 0.08], [0.02, 0.01, 0.013], [2e-3, 3e-3, 1e-3], [2e-4, 1e-4, 3e-4]])
    p.rx_pos = np.r_[p.rx_pos, corner + near]
    p.ris.elems = p.ris.elems[:70].copy()
    p.gamma = p.gamma[:70].copy()
    return p


# 10 708 triangles: lanes per ray below 163 000 rays at order 2, waves above
def test_stacks_fill_at_every_level(ctx):
    base = synth.lab_room_scene(np.random.default_rng(5), sub=7)
    rng = np.random.default_rng(6)
    ext, V, T = np.array([6.0, 5.0, 3.0]), [base.V.astype(np.float64)], [base.T]
    n = len(base.V)
    for i in range(40):   # element i: Morton code 2^(62 - i) and the seven codes after it
        for j in range(8):
            q = np.array([j >> 2, j >> 1 & 1, j & 1], float) + 0.5
            q[i % 3] += 2.0 ** (20 - i // 3)
            u, v = synth.unit(rng.normal(size=3)), 0.7 * synth.unit(rng.normal(size=3))
            V.append(q * ext / 2.0 ** 21 + np.stack([u, v, -u - v]))   # the centroid at the cell's centre
            T.append(np.array([[n, n + 1, n + 2]]))
            n += 3
    nt = sum(len(t) for t in T)
    print("case deep stacks", nt, flush=True)
    p = _problem(_scene(V, T, [np.arange(nt)], 1), np.zeros(3))
    _equals_brute_force(ctx, p, (40, 63), (20_000, 200_000))


def _chain(n, ext, first, d=1e-6):
    """Tiny triangles of one surface in the plane z = 0, element i in the Morton
    cell of bit `first` + i of x and y in turn, the last ones near (0, 0)."""
    V = []
    for i in range(n):
        q = np.array([0.5, 0.5])
        q[i % 2] += 2.0 ** (20 - first - i // 2)
        c = np.r_[q * ext[:2] / 2.0 ** 21, 0.0]
        V.append(c + d * np.array([[1.0, 0.0, 0.0], [-0.5, 0.866, 0.0], [-0.5, -0.866, 0.0]]))
    return np.concatenate(V), np.arange(3 * n).reshape(n, 3)


def test_deep_subtree_of_a_surface(ctx):
    base = synth.lab_room_scene(np.random.default_rng(5), sub=3)
    V, T = _chain(38, np.array([6.0, 5.0, 3.0]), 0)
    print("case deep surface", flush=True)
    scene = _scene([base.V, V], [base.T, T + len(base.V)], [base.surf, np.full(len(T), base.surf.max() + 1)], 2)
    _equals_brute_force(ctx, _problem(scene, np.zeros(3)), (38, 63), (5_000, 100_000))


@pytest.mark.parametrize("first", [0, 1])
def test_split_tree_too_deep(ctx, first):
    """8006 surfaces, most of 17 triangles, and one with a subtree of more than 50
    levels: a chain, and triangles of one Morton cell that only their indices (0
    and the powers of two) tell apart.  The linear BVH of the scene shares the
    chain's upper levels with the other surfaces (59 and 61 levels), the split above
    the surfaces adds its own: 62 levels, and 65, more than the stacks hold."""
    rng = np.random.default_rng(3)
    ext = np.array([12.0, 10.0, 3.0])
    room = synth.box_room(tuple(ext), 0.5 + 0j, sub=2)
    V, T, surf = [room.V], [room.T], [room.surf]
    n, s = len(room.V), 6
    for _ in range(8000):
        axis = int(rng.integers(3))
        u, v = (axis + 1) % 3, (axis + 2) % 3
        a = 2 * np.pi * np.arange(19) / 19 + 0.3
        q = np.repeat(rng.uniform((1.0, 1.0, 0.3), (11.5, 9.5, 2.8))[None], 19, 0)
        h = rng.uniform(0.02, 0.2, 2)
        q[:, u] += h[0] * np.cos(a)
        q[:, v] += h[1] * np.sin(a)
        V.append(q)
        T.append(n + np.c_[np.zeros(17, int), np.arange(1, 18), np.arange(2, 19)])
        surf.append(np.full(17, s))
        n, s = n + 19, s + 1
    cv, ct = _chain(38, ext, first)
    tv = np.concatenate([np.r_[0.5 * ext[:2] / 2.0 ** 21, 0.0] + 1e-6 * (1 + 0.05 * k) *
                         np.array([[1.0, 0.0, 0.0], [-0.5, 0.866, 0.0], [-0.5, -0.866, 0.0]]) for k in range(19)])
    V += [cv, tv]
    T += [ct + n, np.arange(57).reshape(19, 3) + n + len(cv)]
    surf.append(np.full(len(ct) + 19, s))
    T, surf = np.concatenate(T), np.concatenate(surf)
    # the 19 last triangles to the indices 0 and the powers of two
    at = [0] + [1 << k for k in range(18)]
    order = np.full(len(T), -1)
    order[at] = len(T) - 19 + np.arange(19)
    order[order < 0] = np.arange(len(T) - 19)
    print("case split tree too deep", first, len(T), flush=True)
    p = _problem(_scene(V, [T[order]], [surf[order]], 4), np.zeros(3))
    p.order = 1
    _equals_brute_force(ctx, p, (55, 63), (3_000,))
