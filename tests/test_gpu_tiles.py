"""Tile distribution of the persistent find: few seeds against many waves,
tiles dealt out statically, claimed and taken from other queues."""
import numpy as np
import pytest

from synth import barrel_endcap, generate

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("n_events,n_tracks", [(1, 400), (3, 300), (9, 40), (150, 6)])
def test_every_seed_is_found_once(n_events, n_tracks):
    """Seed counts around the tile's 10 (and 8) seeds and the 8 queues, events sorted
    alone and in groups (150 events), one
    block per CU (static tiles) and one wave's worth of blocks: the tracks are
    bitwise those of the layer-synchronous form."""
    from paper_1811_04141_amd import mkf
    w = barrel_endcap(n_events, n_tracks)
    b = generate(w)
    ctx = {}
    for form, flags in (("layers", 0), ("batched", mkf.F_BATCHED)):
        c = ctx[form] = mkf.Context(w.find, flags=flags)
        c.load_geometry(w.layers)
        c.load_hits(b.ev_off, dev(b.x), dev(b.y), dev(b.z), dev(b.var_u), dev(b.var_v),
                    dev(b.layer))
    total = b.seed_hits.shape[0]
    pick = np.random.default_rng(3).permutation(total)
    for n in (0, 1, 8, 9, 10, 11, 79, 81, total):
        sel = np.sort(pick[:n])
        se, sh = b.seed_event[sel], b.seed_hits[sel]
        for c in ctx.values():
            c.seed(dev(se), dev(sh))
        ctx["layers"].find()
        ref = ctx["layers"].get_tracks(n)
        steps = ctx["layers"].stats()["n_steps"]
        for shape in ((2, 8, 0), (1, 1, 6), (3, 3, 8)):
            ctx["batched"].set_tuning(*shape)
            for _ in range(2):
                ctx["batched"].find()
                assert ctx["batched"].get_tracks(n).tobytes() == ref.tobytes(), (n, shape)
                assert ctx["batched"].stats()["n_steps"] == steps, (n, shape)
    for c in ctx.values():
        c.close()
