"""The counting builds walk the scene's Morton tree: the work they report for
small fixed rooms is, number for number, that recorded when it was the only
tree.  Walking the tree with the split above the surfaces instead gives fewer
node visits (739 427 for 2 049 132 of the first room's element legs)."""
import pytest

from paper_2402_13034_amd import synth

pytestmark = pytest.mark.gpu


# per-element kernel: node visits, triangle tests, containment tests, pairs, legs; discovery: node visits, triangle
# tests, segments from the transmitter and from the RIS centre
@pytest.mark.parametrize("sub,order,ris,disc", [
    (3, 2, [2049132, 539, 60969, 32258, 82821], [941116, 107376, 40000, 1277262, 116817, 40000]),
    (6, 1, [448939, 0, 22606, 11430, 20828], [558870, 40903, 20000, 677365, 42456, 20000]),
    (1, 3, [4630300, 1721, 168930, 71120, 236284], [1483752, 190707, 59999, 1672572, 207639, 60000])])
def test_recorded_work(sub, order, ris, disc):
    from paper_2402_13034_amd import risrt
    p = synth.lab_room(nx=4, ny=4, sub=sub, n_rays=20_000, order=order)
    print("case counting", sub, order, p.scene.n_tri, flush=True)
    with risrt.Context(0) as ctx:
        scene, r = risrt.upload_problem(ctx, p)
        ch, st = risrt.trace_problem(ctx, p, scene, r, flags=risrt.FLAG_COUNT_WORK)
        for h in (ch, scene, r):
            ctx.destroy(h)
    assert list(st["ris_work"]) == ris and list(st["discovery_work"]) == disc
