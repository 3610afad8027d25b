"""Bodies past a wall in a batch: accepted, stepped with a force window held inside the lattice, and
reported at the next synchronisation."""
import numpy as np
import pytest

from paper_2207_06029_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bc", [I.BC_ZOUHE_VELOCITY, I.BC_BOUNCEBACK])
@pytest.mark.parametrize("lowest", [-20.0, -7.0, 41.0, 53.0, 110.0])   # of the body's nodes 0..8 in 48
def test_a_body_past_a_wall_ends_with_a_domain_error(bc, lowest):
    from paper_2207_06029_amd import _lib as L, api
    kind = [I.BC_PERIODIC] * 6
    kind[2] = kind[3] = bc
    jobs = []
    for at in (lowest, 19.5):
        xyz, tri = I.spheroid_mesh(2, (4.0, 4.0, 4.0), (23.5, at + 4.0, 23.5))
        jobs.append(I.Job("wall", I.LatticeSpec(48, 48, 48, 0.8, bc=tuple(kind)),
                          I.BodySpec(rigid=0, ks0=0.01, kb=0.0, kv=0.0, mass_ratio=2.0), xyz, tri, 4))
    bt = api.Batch(jobs, autotune=True)
    bt.step(4)
    with pytest.raises(L.LbibError) as e:
        bt.sync()
    assert e.value.code == -7
    alone = api.Batch(jobs[1:])   # the same tables without the stray body
    alone.step(4)
    alone.sync()
    assert np.isfinite(alone.lattice(0).macros()[1]).all()
