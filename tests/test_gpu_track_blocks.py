"""The kernels that take one lane per track in blocks of one wavefront: results,
smoothed states and refits do not depend on how many tracks share the call."""
import numpy as np
import pytest

from synth import barrel_endcap, generate

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("flags", [0, 1])
def test_tracks_do_not_depend_on_the_block_they_fall_in(flags):
    from paper_1811_04141_amd import mkf
    w = barrel_endcap(1, 300)
    b = generate(w)
    c = mkf.Context(w.find, flags=flags)
    c.load_geometry(w.layers)
    c.load_hits(b.ev_off, dev(b.x), dev(b.y), dev(b.z), dev(b.var_u), dev(b.var_v), dev(b.layer))

    def run(n):
        c.seed(dev(b.seed_event[:n]), dev(b.seed_hits[:n]))
        c.find()
        k = mkf.MAX_PLAN + 1
        z = [torch.zeros(s, device="cuda") for s in ((n, k, 6), (n, k, 21), (n, 6), (n, 21), (n,))]
        i = [torch.zeros(n, dtype=torch.int32, device="cuda") for _ in range(2)]
        c.smooth(z[0], z[1], i[0])
        c.backward_fit(z[2], z[3], z[4], i[1])
        torch.cuda.synchronize()
        return [c.get_tracks(n)] + [t.cpu().numpy() for t in z + i]

    ref = run(b.seed_hits.shape[0])
    assert (ref[6] > 3).any() and (ref[7] == 1).any()
    for n in (1, 63, 64, 65, 129):
        for got, want in zip(run(n), ref):
            assert got.tobytes() == np.ascontiguousarray(want[:n]).tobytes(), n
    c.close()


@pytest.mark.parametrize("n_cand", [6, 8])
def test_hit_histories_of_every_plan_length(n_cand):
    """Plans that end on, before and behind a group of eight steps: the
    layer-synchronous form, which follows the back-pointers from memory, gives
    bitwise the persistent form's tracks and steps."""
    import dataclasses
    from paper_1811_04141_amd import mkf
    from synth import Region
    w = barrel_endcap(1, 300)
    b = generate(w)
    big = float(np.finfo(np.float32).max)
    order = list(range(len(w.layers)))
    got = {}
    for flags in (0, mkf.F_BATCHED):
        c = mkf.Context(dataclasses.replace(w.find, n_cand=n_cand), flags=flags)
        c.load_geometry(w.layers)
        for steps in (1, 7, 8, 9, 16, 17, 25):
            c.load_steering((Region(-big, big, tuple(order[:steps + 3])),))
            c.load_hits(b.ev_off, dev(b.x), dev(b.y), dev(b.z), dev(b.var_u), dev(b.var_v),
                        dev(b.layer))
            c.seed(dev(b.seed_event), dev(b.seed_hits))
            c.find()
            t = c.get_tracks(b.seed_hits.shape[0])
            assert (t["plan_len"] == steps).any()
            got.setdefault(steps, []).append((t.tobytes(), c.stats()["n_steps"]))
        c.close()
    for steps, (a, p) in got.items():
        assert a == p, steps


def test_smoothing_of_more_tracks_than_one_wavefront_blocks_take():
    """Above 262,144 tracks smoothing runs in blocks of four wavefronts: every
    copy of a seed gets bitwise the states it gets in a call of 257 (a block and
    one lane of either kind)."""
    from paper_1811_04141_amd import mkf
    w = barrel_endcap(1, 300)
    b = generate(w)
    c = mkf.Context(w.find, flags=mkf.F_BATCHED)
    c.load_geometry(w.layers)
    c.load_hits(b.ev_off, dev(b.x), dev(b.y), dev(b.z), dev(b.var_u), dev(b.var_v), dev(b.layer))
    k, m = mkf.MAX_PLAN + 1, 257

    def run(n):
        at = np.arange(n) % m
        c.seed(dev(b.seed_event[:m][at]), dev(b.seed_hits[:m][at]))
        c.find()
        out = [torch.zeros((n, k, 6), device="cuda"), torch.zeros((n, k, 21), device="cuda"),
               torch.zeros(n, dtype=torch.int32, device="cuda")]
        c.smooth(*out)
        torch.cuda.synchronize()
        return out

    ref = run(m)
    for n in (1 << 18, (1 << 18) + 1):
        at = torch.arange(n, device="cuda") % m
        for got, want in zip(run(n), ref):
            assert torch.equal(got.view(torch.int32), want.view(torch.int32)[at]), n
    c.close()
