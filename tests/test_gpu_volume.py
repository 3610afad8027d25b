"""Enclosed volumes, folded from the centroid kernel's partial sums (one per eight triangles) by a
256-thread block that stands in for 512 threads: sizes below, at and above both counts and above the
2048 partials of one load round."""
import os

import numpy as np
import pytest

from paper_2207_06029_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def api():
    from paper_2207_06029_amd import api as A
    return A


def _job(level):
    # the volume penalty is the membrane's only elasticity: a partial sum left out or counted twice
    # changes (V - V0) / V0 from about 1e-5 to at least 1e-3
    spec = I.LatticeSpec(24, 24, 24, 0.8, **I.shear_walls(0.01))
    xyz, tri = I.spheroid_mesh(level, (3.6, 3.4, 3.1), (11.6, 11.4, 11.7))
    return I.Job("volume", spec, I.BodySpec(rigid=0, ks0=0.0, kb=0.0, kv=1.0, mass_ratio=2.0), xyz, tri, 5)


@pytest.mark.parametrize("level", [1, 3, 4, 5])   # 10, 160, 640 and 2560 partials
def test_volume_penalty_matches_oracle(api, orc, level):
    """FP32 populations round at 6e-8 of order-one values, of which u* ~ 1e-2 keeps about 1e-6
    relative; displacement and velocity inherit it, the forces an order more."""
    orc.set_threads(max(1, min(16, os.cpu_count() or 1)))
    job = _job(level)
    nx, ny, nz = job.lattice.nx, job.lattice.ny, job.lattice.nz
    rho, u = I.random_fields((nx, ny, nz), seed=4, amp_rho=1e-4, amp_u=5e-3)
    u[0] += np.tile(np.repeat(0.02 * (np.arange(ny) / (ny - 1) - 0.5), nx), nz)
    out = []
    for lat in (api.Lattice(job.lattice), orc.Lattice(job.lattice)):
        lat.init(rho, u)
        b = lat.add_body(job.body, job.xyz, job.tri)
        lat.step(job.steps)
        x, v = lat.body_state(b)
        out.append((lat.macros()[1], x - job.xyz, v, lat.body_forces(b)[0]))
    for got, ref, tol in zip(*out, (2e-6, 5e-6, 5e-6, 5e-5)):
        assert np.linalg.norm(got - ref) <= tol * np.linalg.norm(ref)


def test_volumes_in_a_batch_equal_the_jobs_alone(api):
    jobs = [_job(1), _job(4), _job(3)]
    mix = api.Batch(jobs)
    mix.step(5)
    for j, job in enumerate(jobs):
        alone = api.Batch([job])
        alone.step(5)
        for p, q in zip((*mix.lattice(j).body_state(0), *mix.lattice(j).body_forces(0)),
                        (*alone.lattice(0).body_state(0), *alone.lattice(0).body_forces(0))):
            np.testing.assert_array_equal(p, q)
