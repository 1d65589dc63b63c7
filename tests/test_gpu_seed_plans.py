"""Seed states and layer plans do not depend on how many seeds share a call:
eight lanes per seed in small calls, four in large ones, and blocks that end
within a group of lanes."""
import numpy as np
import pytest

from synth import (barrel_endcap, barrel_endcap_field, barrel_material, cms_like, five_regions,
                   generate)

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("setup", ["plain", "steered", "material", "field"])
def test_states_do_not_depend_on_the_number_of_seeds(setup):
    from paper_1811_04141_amd import mkf
    w = {"plain": barrel_endcap, "steered": cms_like, "material": barrel_material,
         "field": barrel_endcap_field}[setup]()
    b = generate(w, events=[0])
    c = mkf.Context(w.find)
    c.load_geometry(w.layers)
    if setup == "steered":
        c.load_steering(five_regions())
    if setup == "material":
        c.load_material(w.material)
    if setup == "field":
        c.load_field(w.field)
    c.load_hits(b.ev_off, dev(b.x), dev(b.y), dev(b.z), dev(b.var_u), dev(b.var_v), dev(b.layer))
    se, sh = b.seed_event[:61], b.seed_hits[:61]
    c.seed(dev(se), dev(sh))
    ref = c.get_seed_states(61)
    assert ref[2].any() and (ref[3] > 0).any()
    for n in (1, 31, 32, 33, 32768, 32769, 40001):
        at = np.arange(n) % 61
        c.seed(dev(se[at]), dev(sh[at]))
        for x, y in zip(c.get_seed_states(n), ref):
            assert np.ascontiguousarray(x).tobytes() == np.ascontiguousarray(y[at]).tobytes(), n
    c.close()


@pytest.mark.parametrize("material", [False, True])
def test_states_on_both_sides_of_the_lanes_rule(material):
    """24,576 seeds are the last to have eight lanes each."""
    from paper_1811_04141_amd import mkf
    w = barrel_material() if material else barrel_endcap()
    b = generate(w, events=[0])
    c = mkf.Context(w.find)
    c.load_geometry(w.layers)
    if material:
        c.load_material(w.material)
    c.load_hits(b.ev_off, dev(b.x), dev(b.y), dev(b.z), dev(b.var_u), dev(b.var_v), dev(b.layer))
    ref = None
    for n in (61, 24576, 24577):
        at = np.arange(n) % 61
        c.seed(dev(b.seed_event[at]), dev(b.seed_hits[at]))
        got = c.get_seed_states(n)
        ref = got if ref is None else ref
        for x, y in zip(got, ref):
            assert np.ascontiguousarray(x).tobytes() == np.ascontiguousarray(y[at]).tobytes(), n
    c.close()
