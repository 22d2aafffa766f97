"""Discovery on either side of the line between four lanes per ray and a wave
per 64 rays, for every order: hit lists, candidates and segment counts of
testing every triangle."""
import numpy as np
import pytest

from paper_2402_13034_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_2402_13034_amd import risrt
    with risrt.Context(0) as c:
        yield c


# 1908 triangles: the line lies at 43 099 rays for order 1, 82 093 for 2, 133 400 for 3, 246 278 for 4 and 5
@pytest.mark.parametrize("n_rays,order", [(43_000, 1), (43_200, 1), (82_000, 2), (82_200, 2), (133_300, 3), (133_500, 3),
                                          (246_200, 4), (246_400, 4), (246_200, 5)])
def test_equals_brute_force(ctx, n_rays, order):
    from paper_2402_13034_amd import risrt
    p = synth.lab_room(nx=3, ny=3, n_rays=n_rays, order=order)
    assert p.scene.n_tri == 1908
    p.ris.elems = p.ris.elems[:3].copy()
    p.gamma = p.gamma[:3].copy()
    print("case discovery lanes", n_rays, order, flush=True)
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
