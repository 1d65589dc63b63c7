"""Duplicate removal at track counts around the lane group's and the wavefront's
sizes, tracks sharing all, some or none of their hits."""
import numpy as np
import pytest

from synth import generate, small_barrel

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def by_rule(tracks, seed_hits, frac):
    """The rule, pair by pair: t is a duplicate if a track ranking before it (more
    hits, smaller chi2, smaller triplet) shares frac of the shorter's hits."""
    hits = [set(int(h) for h in s) | set(int(h) for h in t["hit"] if h >= 0)
            for t, s in zip(tracks, seed_hits)]
    rank = [(-len(h), float(t["chi2"]), tuple(int(v) for v in s))
            for h, t, s in zip(hits, tracks, seed_hits)]
    out = np.zeros(len(tracks), np.int32)
    for t in range(len(tracks)):
        for u in range(len(tracks)):
            if u != t and rank[u] < rank[t]:
                shared = len(hits[t] & hits[u])
                if shared >= float(np.float32(frac)) * min(len(hits[t]), len(hits[u])) and shared:
                    out[t] = 1
    return out


@pytest.mark.parametrize("n", [1, 2, 7, 8, 9, 63, 65, 257])
@pytest.mark.parametrize("frac", [0.2, 0.5, 1.0])
def test_duplicates_follow_the_rule(n, frac):
    from paper_1811_04141_amd import mkf
    w = small_barrel()
    b = generate(w)
    ev = b.events[0]
    rng = np.random.default_rng(n)
    # seeds of a few tracks: their first three hits, later triplets of the same
    # track, and the same triplet again
    seeds = []
    for t in rng.integers(0, max(2, n // 4), 4 * n):
        h = ev.track_hits[t]
        k = rng.integers(0, len(h) - 2)
        seeds.append(h[k:k + 3])
    seeds = np.array(seeds[:n], np.int32).reshape(-1, 3)
    ctx = mkf.Context(w.find, flags=mkf.F_BATCHED)
    ctx.load_geometry(w.layers)
    ctx.load_hits(b.ev_off, dev(b.x), dev(b.y), dev(b.z), dev(b.var_u), dev(b.var_v),
                  dev(b.layer))
    ctx.seed(dev(np.zeros(n, np.int32)), dev(seeds))
    ctx.find()
    tr = ctx.get_tracks(n)
    assert (tr["status"] == 1).all()
    dup = torch.full((n + 1,), -7, dtype=torch.int32, device="cuda")
    n_dup = ctx.find_duplicates(frac, dup)
    ctx.close()
    got = dup.cpu().numpy()
    assert got[n] == -7 and n_dup == int(got[:n].sum())
    assert (got[:n] == by_rule(tr, seeds, frac)).all()
