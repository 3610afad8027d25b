"""Replayed steps where the calls that the CPU tests of the host code count as replayed run on the GPU:
a long first call, bodies added between two replayed stretches, and a stream that is still busy."""
import numpy as np
import pytest

from paper_2207_06029_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def api():
    from paper_2207_06029_amd import api as A
    return A


def _lattice(api, storage=0, stream=None):
    spec = I.LatticeSpec(24, 20, 24, 0.8, storage=storage, **I.shear_walls(0.01))
    xyz, tri = I.spheroid_mesh(2, (3.0, 3.0, 2.4), (11.6, 9.4, 6.2))
    lat = api.Lattice(spec, stream=stream)
    lat.init(*I.random_fields((24, 20, 24), seed=4, amp_rho=1e-4, amp_u=5e-3))
    body = I.BodySpec(rigid=0, ks0=0.01, kb=0.0, kv=0.0, mass_ratio=2.0)
    lat.add_body(body, xyz, tri)
    return lat, lambda: lat.add_body(body, xyz + np.array([0.0, 0.0, 11.5]), tri)


def _equal(a, b, bodies=1):
    state = lambda l: (*l.macros(), *(v for k in range(bodies) for v in (*l.body_state(k), *l.body_forces(k))))
    for p, q in zip(state(a), state(b)):
        np.testing.assert_array_equal(p, q)


@pytest.mark.parametrize("storage", [0, 1])
def test_a_long_first_call_equals_single_steps(api, storage):
    (a, _), (b, _) = _lattice(api, storage), _lattice(api, storage)
    a.step(3)
    a.step(1100)
    for _ in range(1103):
        b.step(1)
    _equal(a, b)


def test_a_body_between_replayed_stretches(api):
    (a, more_a), (b, more_b) = _lattice(api), _lattice(api)
    for more, bodies in ((more_a, 1), (None, 2)):
        a.step(512)
        a.step(64)
        for _ in range(576):
            b.step(1)
        _equal(a, b, bodies)
        if more:
            assert more_a() == more_b() == 1


def test_a_replay_is_captured_while_the_stream_is_busy(api):
    import torch
    s = torch.cuda.Stream()
    (a, _), (b, _) = _lattice(api, stream=s), _lattice(api)
    a.step(512)
    s.synchronize()
    with torch.cuda.stream(s):
        torch.cuda._sleep(2_000_000_000)   # about a second of the GPU's clock
        slept = torch.cuda.Event()
        slept.record()
    a.step(64)
    assert not slept.query()
    for _ in range(576):
        b.step(1)
    _equal(a, b)
