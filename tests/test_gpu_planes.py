"""Population planes padded to whole lines (library memory) against unpadded ones (a caller's
workspace of exactly the reported size): the same results bit for bit, at node counts around the
alignment, through init, steps, streaming, getters and setters, and for jobs in server slots."""
import numpy as np
import pytest

from paper_2207_06029_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def api():
    from paper_2207_06029_amd import api as A
    return A


@pytest.mark.parametrize("storage", [I.STORE_F32, I.STORE_F16, I.STORE_BF16])
@pytest.mark.parametrize("dims", [(1, 3, 1), (4, 4, 4), (13, 5, 1), (9, 7, 5), (67, 33, 19), (128, 5, 7)])
def test_padded_planes_equal_a_workspace_without_padding(api, dims, storage):
    import torch
    spec = I.LatticeSpec(*dims, 0.8, storage=storage, **I.shear_walls(0.01))
    need = api.workspace_bytes(spec)
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    rho, u = I.random_fields(dims, seed=2)
    out = []
    for lat in (api.Lattice(spec), api.Lattice(spec, workspace_ptr=ws.data_ptr(), workspace_bytes=need)):
        lat.init(rho, u)
        lat.step(7)
        f = lat.populations()
        lat.set_populations(f)
        lat.stream_only(3)
        lat.step(2)
        out.append([f, lat.populations(), *lat.macros(), *lat.macros_noalloc(np.empty(spec.n), np.empty(3 * spec.n))])
        lat.destroy()
    for a, b in zip(*out):
        np.testing.assert_array_equal(a, b)


@pytest.mark.parametrize("slot_nodes", [23 * 21 * 25, 23 * 21 * 25 + 70])
def test_served_job_with_and_without_room_for_padding_equals_the_job_alone(api, slot_nodes):
    spec = I.LatticeSpec(23, 21, 25, 0.8, storage=I.STORE_F16, **I.shear_walls(0.01))
    xyz, tri = I.spheroid_mesh(2, (3.5, 3.5, 3.0), (11.0, 10.0, 12.0))
    body = I.BodySpec(rigid=0, ks0=0.01, kb=0.001, kv=0.0, mass_ratio=1.0)
    job = I.Job("odd", spec, body, xyz, tri, 30)
    srv = api.Server(1 << 30, 2, 10, storage=I.STORE_F16, slot_nodes=slot_nodes, slot_vertices=len(xyz))
    ids = [srv.submit(job) for _ in range(3)]
    done = {}
    while len(done) < len(ids):
        srv.tick()
        done.update({r["id"]: r for r in srv.poll(with_positions=True)})
    alone = api.Batch([job], storage=I.STORE_F16)
    alone.step(30)
    x = alone.lattice(0).body_state(0)[0]
    for i in ids:
        assert done[i]["status"] == 0
        np.testing.assert_array_equal(done[i]["xyz"], x)
