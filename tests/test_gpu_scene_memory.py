"""What a scene holds and what its build needs at once: 628 bytes a triangle
(all surface tables sized for one surface a triangle) and 4 a surface table's
end, and budgets in which scenes from host arrays have always fitted."""
import numpy as np
import pytest

from paper_2402_13034_amd import synth

pytestmark = pytest.mark.gpu


def _scene(name):
    if name == "box":
        return synth.box_room((5.0, 4.0, 3.0), 0.5 + 0j)
    if name.startswith("lab"):
        return synth.lab_room_scene(np.random.default_rng(5), sub=int(name[3:]))
    sc, n = synth.lab_room_scene(np.random.default_rng(5), sub=9), int(name[6:])   # every triangle a surface
    return synth.Scene(sc.V, sc.T[:n].copy(), sc.refl_re[:n].copy(), sc.refl_im[:n].copy(), np.arange(n, dtype=np.int32))


@pytest.mark.parametrize("name,budget", [("box", 16384), ("lab3", 1806336), ("single100", None), ("single2048", None),
                                         ("single8192", 7507968), ("lab9", None)])
def test_bytes_and_budget(name, budget):
    from paper_2402_13034_amd import risrt
    sc = _scene(name)
    print("case scene memory", name, sc.n_tri, flush=True)
    with risrt.Context(0, budget or 0) as ctx:
        h = ctx.scene_create(sc.V, sc.T, sc.surf, sc.refl_re, sc.refl_im)
        assert ctx.scene_info(h)["bytes"] <= 628 * sc.n_tri + 4
        ctx.destroy(h)
