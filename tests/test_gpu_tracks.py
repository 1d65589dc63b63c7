"""Track records handed back to the caller: one chunk, several, and part-filled
ones, in seed order."""
import numpy as np
import pytest

from synth import generate, small_barrel

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

CHUNK = 16384  # records per pinned slot of the library


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("n", [1, 1025, 5000, CHUNK - 1, CHUNK, CHUNK + 1, 20481, 3 * CHUNK - 5,
                               30721, 40960, 40961, 9 * CHUNK + 7])
def test_records_in_seed_order(n):
    """An event's seeds repeated to n: every record is its seed's own, whatever
    the number of chunks and the launch shape the find takes for n seeds, also
    into a longer and into a shorter array."""
    from paper_1811_04141_amd import mkf
    w = small_barrel()
    b = generate(w)
    m = b.seed_hits.shape[0]
    ctx = mkf.Context(w.find, flags=mkf.F_BATCHED)
    ctx.load_geometry(w.layers)
    ctx.load_hits(b.ev_off, dev(b.x), dev(b.y), dev(b.z), dev(b.var_u), dev(b.var_v),
                  dev(b.layer))
    ctx.seed(dev(b.seed_event), dev(b.seed_hits))
    ctx.find()
    one = ctx.get_tracks(m)
    assert (one["status"] == 1).all() and (one["n_hits"] > 3).all()
    k = np.arange(n) % m
    ctx.seed(dev(b.seed_event[k]), dev(b.seed_hits[k]))
    ctx.find()
    want = one[k].copy()
    want["seed_id"] = np.arange(n)
    assert ctx.get_tracks(n).tobytes() == want.tobytes()
    more = ctx.get_tracks(n + 3)
    assert more[:n].tobytes() == want.tobytes() and not any(more[n:].tobytes())
    short = np.full(n + 1, 0, mkf.TRACK_DTYPE)
    total = mkf.C.c_int64()
    st = mkf.lib.mkf_get_tracks(ctx.h, mkf.C.c_void_p(short.ctypes.data), max(0, n - 1),
                                mkf.C.byref(total))
    assert st == mkf.MKF_E_CAPACITY and total.value == n
    assert short[:n - 1].tobytes() == want[:n - 1].tobytes() and not any(short[n - 1:].tobytes())
    ctx.close()
