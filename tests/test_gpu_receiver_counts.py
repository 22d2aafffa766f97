"""Receivers by the thousand: where the counts per receiver go from one
workgroup's scan to the tiled one and from one stretch of 8192 to the next, the
order by position begins and takes more bits, and the centre's sequences come out of one
wave per receiver.  Every receiver's result is that of a trace with a few of
them, whatever the others are."""
import numpy as np
import pytest

from paper_2402_13034_amd import synth

pytestmark = pytest.mark.gpu
PART = 700


@pytest.fixture(scope="module")
def ctx():
    from paper_2402_13034_amd import risrt
    with risrt.Context(0) as c:
        yield c


def _trace(ctx, prob, flags):
    from paper_2402_13034_amd import risrt
    scene, ris = risrt.upload_problem(ctx, prob)
    ch, st = risrt.trace_problem(ctx, prob, scene, ris, flags=flags)
    E, H = ctx.channel_read(ch)
    p = ctx.paths_read(ch) if flags else None
    for h in (ch, scene, ris):
        ctx.destroy(h)
    return E, H, st, p


# unsorted up to 256; R + 1 counts: a stretch of 4096 less one, a full one, one more, two, then around the limit of
# one workgroup's scan, 16384, and twice that
@pytest.mark.parametrize("n_rx", [1, 65, 256, 257, 4094, 4095, 4096, 8191, 8192, 16382, 16383, 16384, 32768])
def test_receivers_do_not_touch_each_other(ctx, n_rx):
    from paper_2402_13034_amd import risrt
    p = synth.lab_room(nx=4, ny=4, n_rays=20_000, order=2)
    p.ris.elems = p.ris.elems[:5].copy()
    p.gamma = p.gamma[:5].copy()
    rng = np.random.default_rng(n_rx)
    # a third in one corner, some outside the room, the rest over it
    rx = rng.uniform((0.2, 0.2, 0.2), (5.8, 4.8, 2.8), (n_rx, 3))
    rx[::3] = 1.0 + 0.01 * rx[::3]
    rx[5::11] += 7.0
    p.rx_pos = rx
    print("case receivers", n_rx, flush=True)
    E, H, st, _ = _trace(ctx, p, 0)
    Ek, Hk, stk, kept = _trace(ctx, p, risrt.FLAG_KEEP_PATHS)
    assert np.array_equal(E, Ek) and np.array_equal(H, Hk)
    assert st["n_env_paths"] == stk["n_env_paths"] == len(kept["env"])
    assert st["n_u_paths"] == stk["n_u_paths"]
    n_env = n_u = 0
    for a in range(0, n_rx, PART):
        p.rx_pos = rx[a:a + PART].copy()
        e, h, s, _ = _trace(ctx, p, 0)
        n_env += s["n_env_paths"]
        n_u += s["n_u_paths"]
        assert np.array_equal(E[a:a + PART], e) and np.array_equal(H[a:a + PART], h)
    assert (st["n_env_paths"], st["n_u_paths"]) == (n_env, n_u)
