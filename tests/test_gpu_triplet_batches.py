"""Triplet seeding of batches whose events differ in size."""
import time

import numpy as np
import pytest

from synth import SeedingConfig, barrel_endcap, generate_event

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

FIELDS = ("x", "y", "z", "var_u", "var_v", "layer")


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def batch(events):
    off = np.concatenate([[0], np.cumsum([len(e.x) for e in events])])
    return off, [dev(np.concatenate([getattr(e, f) for e in events])) for f in FIELDS]


class Seeder:
    def __init__(self, w, cap=1 << 20):
        from paper_1811_04141_amd import mkf
        self.ctx = mkf.Context(w.find)
        self.ctx.load_geometry(w.layers)
        self.ev = torch.empty(cap, dtype=torch.int32, device="cuda")
        self.hits = torch.empty((cap, 3), dtype=torch.int32, device="cuda")
        self.cap = cap

    def load(self, events):
        off, arrs = batch(events)
        self.ctx.load_hits(off, *arrs)

    def seeds(self):
        n = self.ctx.make_seeds(SeedingConfig(), self.cap, self.ev, self.hits)
        t = torch.cat([self.ev[:n, None], self.hits[:n]], 1).cpu().numpy()
        return t[np.lexsort(t.T[::-1])]

    def ms(self, cuts=SeedingConfig()):
        best = 1e30
        for _ in range(8):
            torch.cuda.synchronize()
            t = time.perf_counter()
            self.ctx.make_seeds(cuts, self.cap, self.ev, self.hits)
            best = min(best, time.perf_counter() - t)
        return best * 1e3


@pytest.mark.parametrize("sizes", [(1500, 2000), (300, 3), (0, 1), (0, 7)])
def test_large_event_among_small_ones(sizes):
    """One event of many tracks and many of five, the large one first, last and
    between: each event's triplets are those it has alone."""
    tracks, n_small = sizes
    w = barrel_endcap()
    big = [generate_event(w, 0, n_tracks=tracks)] if tracks else []
    small = generate_event(w, 1, n_tracks=5)
    s = Seeder(w)
    alone = []
    for e in big + [small]:
        s.load([e])
        alone.append(s.seeds()[:, 1:])
    for at in sorted({0, n_small // 2, n_small}):
        events = [small] * n_small
        events[at:at] = big
        s.load(events)
        got = s.seeds()
        want = [np.column_stack([np.full(len(a), e), a])
                for e in range(len(events)) for a in [alone[0 if events[e] is not small else -1]]]
        assert np.array_equal(got, np.concatenate(want))
    s.ctx.close()


def test_large_event_costs_little_more_among_small_ones():
    """An event of 3,000 tracks among 2,000 of five takes at most four times as long
    as alone and the others without it (9.6 times when every event got the same
    share of the wavefronts whatever its size, 1.3 now)."""
    w = barrel_endcap()
    big, small = generate_event(w, 0, n_tracks=3000), generate_event(w, 1, n_tracks=5)
    s = Seeder(w)
    ms = []
    for events in ([big], [small] * 2000, [big] + [small] * 2000):
        s.load(events)
        ms.append(s.ms())
    s.ctx.close()
    assert ms[2] < 4.0 * (ms[0] + ms[1]), ms


def test_small_events_use_the_whole_device():
    """2,000 events of five tracks take about as long as 1,800.  (Twice as long when
    2,000 got eight blocks per event, of which the first two have hits and always
    ran on the same two XCDs, and 1,800 nine.)"""
    w = barrel_endcap()
    small = generate_event(w, 1, n_tracks=5)
    s = Seeder(w)
    ms = []
    for n in (1800, 2000):
        s.load([small] * n)
        ms.append(s.ms())
    s.ctx.close()
    assert ms[1] < 1.5 * ms[0], ms


LOOSE = SeedingConfig(d0_max=1.0)


def test_loose_cuts_on_dense_events():
    """Hundreds of candidates per pair, most of which fail: the set is the one that
    the exact cuts leave of any larger bound, here of d0_max 1.05."""
    from oracle import oracle as O
    w = barrel_endcap()
    e = generate_event(w, 0, n_tracks=1200, phi_range=(0.0, 1.0))
    s = Seeder(w)
    s.load([e])
    got = {}
    for d0 in (1.0, 1.05):
        n = s.ctx.make_seeds(SeedingConfig(d0_max=d0), s.cap, s.ev, s.hits)
        got[d0] = {tuple(h) for h in s.hits[:n].cpu().numpy().tolist()}
        assert len(got[d0]) == n
    s.ctx.close()
    assert got[1.0] < got[1.05]
    for t in sorted(got[1.05] - got[1.0]):
        xyz = [[e.x[i], e.y[i], e.z[i]] for i in t]
        assert O.triplet_params(w.find, LOOSE, *xyz)[1] < 1e-9
    for t in sorted(got[1.0])[::37]:
        xyz = [[e.x[i], e.y[i], e.z[i]] for i in t]
        assert O.triplet_params(w.find, LOOSE, *xyz)[1] > -1e-9


def test_loose_cuts_cost_by_the_candidates():
    """d0_max 1 cm against 0.1 widens the windows and leaves far more candidates to
    the exact cuts.  (89 times as long when walks were repeated for every four
    candidates of a pair, 14 now.)"""
    w = barrel_endcap()
    s = Seeder(w)
    s.load([generate_event(w, 0, n_tracks=3000)])
    ms = [s.ms(), s.ms(LOOSE)]
    s.ctx.close()
    assert ms[1] < 35.0 * ms[0], ms
