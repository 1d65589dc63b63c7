"""The library's host code against a runtime of two devices whose kernels do
nothing (fake_hip.c): which device its calls are made on, what it allocates and
what it launches.  CPU only; each test is a process of its own, so that the
runtime is there before the library."""
import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))

PRELUDE = """
import ctypes as C, sys
fake = C.CDLL(sys.argv[1], C.RTLD_GLOBAL)
fake.fake_launches.restype = fake.fake_wrong_what.restype = C.c_char_p
import numpy as np
from paper_1811_04141_amd import mkf
from synth import generate, small_barrel
w = small_barrel()
b = generate(w)

def context(n, flags=mkf.F_BATCHED, device=0):
    '''A context of `device` with an event's seeds, repeated to n.'''
    ctx = mkf.Context(w.find, flags=flags, stream=0x1000 + device)
    ctx.load_geometry(w.layers)
    ctx.load_hits(b.ev_off, b.x, b.y, b.z, b.var_u, b.var_v, b.layer)
    seed(ctx, n)
    return ctx

def seed(ctx, n):
    k = np.arange(n) % b.seed_hits.shape[0]
    ctx.seed(np.ascontiguousarray(b.seed_event[k]), np.ascontiguousarray(b.seed_hits[k]))
    ctx.find()

def launches():
    out = fake.fake_launches().decode().splitlines()
    fake.fake_reset()
    return out
"""


@pytest.fixture(scope="module")
def fake(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("fake") / "fake_hip.so")
    subprocess.run(["gcc", "-O1", "-std=c11", "-shared", "-fPIC", "-Wall", "-Werror", "-o", so,
                    os.path.join(HERE, "fake_hip.c")], check=True)
    return so


def run(fake, body):
    r = subprocess.run([sys.executable, "-c", PRELUDE + body, fake], cwd=os.path.dirname(HERE),
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr


@pytest.mark.parametrize("n", [200, 40000])
def test_tracks_are_fetched_on_the_contexts_device(fake, n):
    """Records of one slot and of several, with another device current at the
    call than at mkf_create: everything happens on the context's device, and
    the caller's is current again afterwards."""
    run(fake, f"""
ctx = context({n})
assert fake.fake_wrong() == 0, fake.fake_wrong_what()
fake.fake_reset()
fake.hipSetDevice(1)
ctx.get_tracks({n})
assert fake.fake_wrong() == 0, fake.fake_wrong_what()
assert len(launches()) >= 1
d = C.c_int(-1)
fake.hipGetDevice(C.byref(d))
assert d.value == 1
""")


def test_growing_calls_pin_each_slot_once(fake):
    """Events of slowly growing size: a small first slot, then the whole of it,
    then the other seven as calls need them; nothing is pinned again."""
    run(fake, """
ctx = context(200)
fake.fake_reset()
for n in range(100, 1025, 77):
    seed(ctx, n)
    ctx.get_tracks(n)
assert fake.fake_pinned() == 1, fake.fake_pinned()
for n in list(range(1100, 16385, 407)) + [16384]:
    seed(ctx, n)
    ctx.get_tracks(n)
assert fake.fake_pinned() == 2, fake.fake_pinned()
for n in (16385, 30000, 60000, 200000, 150000, 50):
    seed(ctx, n)
    ctx.get_tracks(n)
assert fake.fake_pinned() <= 2 + 7, fake.fake_pinned()
""")


@pytest.mark.parametrize("n", [200, 25000, 40000, 100000])
def test_a_tuning_read_and_set_back_keeps_the_launch(fake, n):
    """mkf_get_tuning's values set back, as they are or with other bins, leave the
    find's launch as it was: by the number of seeds where no shape was set, and
    the shape that was set where one was."""
    run(fake, f"""
def find_launch():
    fake.fake_reset()
    ctx.find()
    return [l for l in launches() if "k_find_persistent" in l]

ctx = context({n})
own = find_launch()
assert len(own) == 1
t = ctx.get_tuning()
ctx.set_tuning(**t)
assert find_launch() == own and ctx.get_tuning() == t
ctx.set_tuning(**dict(t, phi_bin_shift=1))
assert find_launch() == own
ctx.set_tuning(1, 1)
one = find_launch()
assert one != own
ctx.set_tuning(**dict(ctx.get_tuning(), q_bin_shift=-1))
assert find_launch() == one
ctx.set_tuning(2, 8)  # set after another: as it is
two = find_launch()
seed(ctx, 200000)
big = find_launch()
assert "ILi2E" in two[0] and "ILi2E" in big[0] and big[0].split()[1] == "2048"
""")
