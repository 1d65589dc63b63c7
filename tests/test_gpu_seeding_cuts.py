"""Triplet seeding away from the usual cuts: the bounds that drop candidates
before the exact cuts never drop one that passes, whatever the cuts, the number
of triplets per hit and the room to keep them."""
from dataclasses import replace

import numpy as np
import pytest

from oracle import oracle as O
from synth import SeedingConfig, barrel_endcap, generate_event, make_batch

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


CUTS = [SeedingConfig(), SeedingConfig(d0_max=1e-3, dz_max=2e-3),
        SeedingConfig(pt_min=0.05, d0_max=1.5, z0_max=500.0, dz_max=1.5),
        SeedingConfig(pt_min=1.0, d0_max=5.0, z0_max=500.0, dz_max=0.02),
        SeedingConfig(layers=(1, 4, 8), pt_min=0.6, d0_max=0.5, dz_max=3.0, z0_max=500.0),
        SeedingConfig(layers=(0, 5, 6), d0_max=0.05, dz_max=10.0, z0_max=500.0)]


@pytest.mark.parametrize("sc", CUTS)
@pytest.mark.parametrize("phi", [None, (0.0, 0.15), (3.05, 3.2)])
def test_triplets_match_brute_force(sc, phi):
    """Two events of 70 tracks, over the whole azimuth, as a jet (hundreds of
    triplets per first hit) and as a jet across the azimuth's end; the capacity
    is ample, then just enough.  With one bin per layer the search windows hold
    every hit (they are sized for cuts around the usual ones), so the set is the
    brute force's; with the usual bins it is a part of it."""
    from paper_1811_04141_amd import mkf
    w = barrel_endcap()
    evs = [generate_event(w, e, n_tracks=70, phi_range=phi) for e in range(2)]
    b = make_batch(evs)
    want = None
    ctx = mkf.Context(w.find)
    for cap, bins in ((1 << 20, 1), (0, 1), (1 << 20, 0)):
        ctx.load_geometry([replace(L, n_phi_bins=1, n_q_bins=1) if bins else L for L in w.layers])
        ctx.load_hits(b.ev_off, dev(b.x), dev(b.y), dev(b.z), dev(b.var_u), dev(b.var_v),
                      dev(b.layer))
        cap = cap or len(want)
        ev = torch.full((cap + 1,), -7, dtype=torch.int32, device="cuda")
        hits = torch.full((cap + 1, 3), -7, dtype=torch.int32, device="cuda")
        n = ctx.make_seeds(sc, cap, ev, hits)
        assert int(ev[n]) == -7 and int(hits[n, 0]) == -7
        ev, hits = ev[:n].cpu().numpy(), hits[:n].cpu().numpy()
        assert (np.diff(ev) >= 0).all()
        got = sorted((int(e),) + tuple(int(x) for x in h) for e, h in zip(ev, hits))
        assert len(set(got)) == n
        want = got if want is None else want
        assert got == want if bins else set(got) <= set(want)
    ctx.close()
    for e in range(2):
        o, frag, _ = O.triplet_seeds(w.find, sc, evs[e])
        gs, os_ = {t[1:] for t in want if t[0] == e}, {tuple(t) for t in o.tolist()}
        fragile = {tuple(t) for t, f in zip(o.tolist(), frag) if f}
        assert not (os_ - gs - fragile), len(os_ - gs)
        for t in gs - os_:
            xyz = [[evs[e].x[i], evs[e].y[i], evs[e].z[i]] for i in t]
            assert O.triplet_params(w.find, sc, *xyz)[1] > -1e-9
