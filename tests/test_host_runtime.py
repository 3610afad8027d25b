"""The library's host code on the CPU, under a stand-in for the HIP runtime (hip_stub.hip) that runs no
kernel and logs what is asked of it: the tables that the launches get, and when steps are replayed."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# In a process of its own: the stand-in is loaded first and globally, so the library's calls go to it.
# torch stays out (it brings the real runtime).
PREAMBLE = """
import ctypes, sys
sys.modules["torch"] = None
sys.path.insert(0, {root!r})
stub = ctypes.CDLL({stub!r}, mode=ctypes.RTLD_GLOBAL)
stub.stub_log.restype = ctypes.c_char_p
import numpy as np
from paper_2207_06029_amd import api, inputs as I

def log():
    lines = stub.stub_log().decode().splitlines()
    stub.stub_clear()
    return lines

def lattice(n=24, stream=4711):
    lat = api.Lattice(I.LatticeSpec(n, n, n, 0.8, **I.shear_walls(0.01)), stream=stream)
    xyz, tri = I.spheroid_mesh(1, (3.5, 3.5, 2.8), ((n - 1) / 2,) * 3)
    body = I.BodySpec(rigid=0, ks0=0.01, kb=0.0, kv=0.0, mass_ratio=2.0)
    lat.add_body(body, xyz, tri)
    log()
    return lat, lambda: lat.add_body(body, xyz, tri)

def steps(lines, stream=4711):
    "Steps run by these calls, one by one and in replays of 16."
    single = sum("k_sweep" in l and l.endswith(f" {{stream}}") for l in lines)
    return single, 16 * lines.count(f"replay {{stream}}")
"""


@pytest.fixture(scope="module")
def stub(tmp_path_factory):
    from paper_2207_06029_amd import build as B
    so = str(tmp_path_factory.mktemp("stub") / "libhip_stub.so")
    r = subprocess.run([B.HIPCC, "--offload-host-only", "-O1", "-std=c++17", "-shared", "-fPIC", "-w", "-I", B.CSRC,
                        os.path.join(ROOT, "tests", "hip_stub.hip"), "-o", so], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return so


def _run(stub, code):
    r = subprocess.run([sys.executable, "-c", PREAMBLE.format(root=ROOT, stub=stub) + code], capture_output=True, text=True,
                       timeout=300)
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-4000:]


WINDOWS = """
# a body beside, across and beyond either wall of axis a, and anywhere along a periodic axis; the tuner
# sweeps with the layouts that the host wrote
n = 48
for a in range(3):
    for at in (-1e12, -60.0, -9.0, -1.5, 0.0, 5.0, 23.5, 47.0, 48.5, 57.0, 64.0, 114.0, 1e9, 1e12):
        for bc in (I.BC_PERIODIC, I.BC_ZOUHE_VELOCITY, I.BC_BOUNCEBACK):
            for rigid in (0, 1):
                kind = [I.BC_PERIODIC] * 6
                kind[2 * a] = kind[2 * a + 1] = bc
                spec = I.LatticeSpec(n, n, n, 0.8, bc=tuple(kind))
                body = I.BodySpec(rigid=rigid, ks0=0.0 if rigid else 0.01, kb=0.0, kv=0.0, mass_ratio=2.0)
                centre = [23.5] * 3
                centre[a] = at
                # far away no mesh keeps its shape in double: only the coordinates' range matters there
                xyz, tri = I.spheroid_mesh(1, (4.0, 4.0, 4.0), (23.5,) * 3)
                xyz[:, a] += at - 23.5
                try:
                    b = api.Batch([I.Job("wall", spec, body, xyz, tri, 1)], autotune=True)
                except Exception as e:
                    assert abs(at) >= 1e9 and "outward" in str(e), (a, at, bc, rigid, e)
                    log()
                    continue
                b.step(1)
                lines = log()
                assert any("k_sweep" in l for l in lines)
                assert not any(l.startswith("bad window") for l in lines), (a, at, bc, rigid)
                b.destroy()
"""


def test_windows_of_bodies_past_a_wall_stay_in_the_lattice(stub):
    """Batches take any body (a support on a wall is reported at the next synchronisation), and the sweep
    reads the force window without testing its layout."""
    _run(stub, WINDOWS)


def test_steps_are_replayed_without_a_wait(stub):
    """Stepping is asynchronous: nothing is waited for where steps are captured and replayed."""
    _run(stub, """
lat, _ = lattice()
lat.step(512)
assert steps(log()) == (512, 0)
# a replay starts on an even step: single steps up to it, and for what is left over
for n, single, replayed in ((15, 15, 0), (64, 16, 48), (16, 16, 0), (35, 3, 32), (16, 0, 16)):
    lat.step(n)
    lines = log()
    assert steps(lines) == (single, replayed), (n, steps(lines))
    assert not any(l.startswith("sync") for l in lines)
""")


def test_a_change_of_the_bodies_ends_the_replays(stub):
    """The graph of the old tables is given up once its replays have ended, and a new one is captured."""
    _run(stub, """
lat, again = lattice()
lat.step(512)
lat.step(64)
assert steps(log()) == (512, 64)
again()
lines = log()
assert lines.count("exec_destroy") == 1 and "exec_destroy busy" not in lines
lat.step(511)
lat.step(65)
assert steps(log()) == (576, 0)
lat.step(64)
lines = log()
assert steps(lines) == (0, 64) and sum(l.startswith("begin") for l in lines) == 1
assert not any(l.startswith("sync") for l in lines)
""")


def test_steps_under_another_device_are_not_replayed(stub):
    """Launches go to their stream's device whichever is current; a graph would be captured for, and
    launched on, the current one."""
    _run(stub, """
lat, _ = lattice()
lat.step(512)
stub.stub_set_device(1)
lat.step(64)
lines = log()
assert steps(lines) == (576, 0) and not any(l.startswith("begin") for l in lines)
stub.stub_set_device(0)
lat.step(64)
assert steps(log()) == (0, 64)
stub.stub_set_device(1)
lat.step(64)
assert steps(log()) == (64, 0)
""")


def test_destroying_a_lattice_waits_for_its_replays(stub):
    """On the default stream too, and for the lattice's device where another one is current."""
    _run(stub, """
for stream in (4711, None):
    for current in (0, 1):
        lat, _ = lattice(stream=stream)
        lat.step(512)
        lat.step(64)
        assert steps(log(), stream or 0) == (512, 64)
        stub.stub_set_device(current)
        lat.destroy()
        lines = log()
        assert lines.count("exec_destroy") == 1 and "exec_destroy busy" not in lines
        stub.stub_log_device()
        assert log() == [f"device {current}"]
        stub.stub_set_device(0)
""")


def test_a_long_first_call_is_replayed_after_its_first_steps(stub):
    _run(stub, """
# steps of calls on a new lattice: (single, replayed) of each
for calls, want in ((((2048,), [(512, 1536)])), ((1024,), [(512, 512)]), ((1023, 17), [(1023, 0), (1, 16)]),
                    ((3, 1100, 16), [(3, 0), (509 + 15, 576), (16, 0)]), ((511, 65, 64), [(511, 0), (65, 0), (0, 64)])):
    lat, _ = lattice()
    got = []
    for n in calls:
        lat.step(n)
        got.append(steps(log()))
    assert got == want, (calls, got)
    assert lat.step_count == sum(calls)
""")


def test_sweep_tiles_in_the_order_of_the_chunk(stub):
    """Blocks go to XCD bid % 8: in every whole turn each takes its own run of `chunk` tiles in order, for
    any chunk of a tuning line, and every tile is taken once."""
    _run(stub, """
for T in (1, 7, 24, 63, 64, 65, 128, 200, 1000):
    for chunk in (0, 1, 2, 3, 5, 8, 13, 25, 125, 126, 1 << 29, 2**31 - 1):
        order = [stub.stub_sweep_tile(T, bid, chunk) for bid in range(T)]
        assert sorted(order) == list(range(T)), (T, chunk)
        turns = T // (8 * chunk) if chunk else 0
        for turn in range(turns):
            for xcd in range(8):
                at = 8 * chunk * turn
                got = order[at + xcd:at + 8 * chunk:8]
                assert got == list(range(at + xcd * chunk, at + (xcd + 1) * chunk)), (T, chunk)
        assert order[8 * chunk * turns:] == list(range(8 * chunk * turns, T))
""")


def test_a_refused_body_leaves_the_lattice_as_it_was(stub):
    """A body that a caller's workspace cannot hold is refused; steps after it run the bodies that were
    there before, and no kernel for the one that was not."""
    _run(stub, """
spec = I.LatticeSpec(24, 24, 24, 0.8, **I.shear_walls(0.01))
xyz, tri = I.spheroid_mesh(1, (3.5, 3.5, 2.8), (11.5,) * 3)
body = I.BodySpec(rigid=0, ks0=0.01, kb=0.0, kv=0.0, mass_ratio=2.0)
for bodies in (0, 1):
    need = api.workspace_bytes(spec, len(xyz) * bodies, len(tri) * bodies) + 4096
    buf = ctypes.create_string_buffer(need + 256)
    lat = api.Lattice(spec, stream=4711, workspace_ptr=(ctypes.addressof(buf) + 255) // 256 * 256, workspace_bytes=need)
    if bodies:
        lat.set_velocity(lat.add_body(body, xyz, tri), np.full(3 * len(xyz), 0.25))
    before = [lat.body_state(b) for b in range(bodies)]
    try:
        lat.add_body(body, xyz, tri)
        assert False
    except Exception as e:
        assert "workspace too small" in str(e)
    log()
    lat.step(2)
    names = {l.split()[1] for l in log()}
    assert any("k_sweep" in n for n in names)
    assert any("k_centroids" in n for n in names) == (bodies == 1)
    for b in range(bodies):
        for p, q in zip(before[b], lat.body_state(b)):
            assert (p == q).all()
    try:
        lat.body_state(bodies)
        assert False
    except Exception as e:
        assert "no such body" in str(e)
""")
