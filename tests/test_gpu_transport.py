"""Edges of the transport's launch: how many started photons a wavefront keeps
in LDS, and photons that miss the phantom."""
import sys

import numpy as np
import pytest

from paper_1204_6367_amd import workloads as W

from test_gpu_materials import sixteen_material_problem

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1204_6367_amd import api
    return api


@pytest.mark.parametrize("macro, interp", [(0, True), (4, True), (4, False)])
@pytest.mark.parametrize("n_e", [299, 1023])
def test_tallies_do_not_depend_on_started_photons_kept(gpu, macro, interp, n_e):
    """16 materials on 1023 energies nearly fill the LDS, so that wide workgroups keep
    16 or 32 started photons a wavefront instead of 64; photon counts that end in
    the middle of a wavefront, and an off-axis detector that most photons reach
    without entering the phantom.  The integer tallies are bit for bit the same."""
    import torch
    prob = sixteen_material_problem(1, shape=(9, 11, 12))
    grid = W.EnergyGrid(de_kev=0.5 * 298 / (n_e - 1), n_e=n_e)
    mu = np.stack([np.stack([np.interp(grid.energies(), W.EnergyGrid().energies(), prob.physics.mu_mass[m, :, k])
                             for k in range(3)], -1) for m in range(16)]).astype(np.float32)
    prob.physics = W.Physics(mu, grid, None)
    vol, phys, src = gpu.upload(prob)
    if macro:
        vol.local_majorants(macro)
    jobs = [gpu.JobSpec(prob.geom.replace(phi_rad=0.9 * k), n, k) for k, n in enumerate((1, 63, 64, 65, 5003, 20_001))]
    b = gpu.Batch([vol], phys, [src], jobs)
    ref = b.project(seed=3, interp=interp, tune=dict(block=64, chunk=64))
    assert float(ref.sum()) > 0
    for t in (None, dict(block=512, defer=1), dict(block=1024, defer=8, chunk=128), dict(block=1024, blocks_per_cu=1)):
        print("shape", t, flush=True)
        assert torch.equal(b.project(seed=3, interp=interp, tune=t), ref), t


@pytest.mark.parametrize("interp", [True, False])
def test_padded_grid_walks_as_the_plain_one(gpu, interp):
    """Cube records staged in the padded LDS grid (all-local launches) and in the plain one
    (a second, single-majorant volume in the launch) give the same histories: single cubes
    along an axis, last cubes shorter than the others, one slab, and lines that leave
    through every face."""
    import torch
    rng = np.random.default_rng(8)
    for shape, macro in (((6, 7, 5), 3), ((4, 4, 4), 4), ((3, 20, 2), 1), ((9, 3, 30), 2), ((2, 60, 70), 2)):
        mat = rng.integers(0, 3, shape).astype(np.uint8)
        dens = rng.uniform(0.05, 2.0, shape).astype(np.float32)
        ph = W.Phantom(dens, mat, (7.0, 6.0, 5.0), ["air", "soft_tissue", "bone"])
        geom = W.Geometry(nu=24, nv=18, du_mm=6.0, dv_mm=6.0)
        prob = W.Problem(ph, W.physics_for(ph), W.pelvis_source(geom), geom, 1)
        vol, phys, src = gpu.upload(prob)
        vol.local_majorants(macro)
        plain = gpu.DeviceVolume(dens, mat, ph.spacing_mm)
        jobs = [gpu.JobSpec(geom.replace(phi_rad=0.7 * k), 20_000, k) for k in range(5)]
        ref = gpu.Batch([vol], phys, [src], jobs).project(seed=5, interp=interp)
        mixed = gpu.Batch([vol, plain], phys, [src], jobs + [gpu.JobSpec(geom, 64, 9, volume=1)])
        got = mixed.project(seed=5, interp=interp)
        if interp:      # (the plain walk is set up afresh for the second flight of a pair)
            same = (got[:ref.numel()] == ref).double().mean()
            assert float(same) > 0.99, float(same)
            assert abs(float(got[:ref.numel()].sum() / ref.sum()) - 1.0) < 1e-3
        else:
            assert torch.equal(got[:ref.numel()], ref), (shape, macro)


def project_with(gpu, b, spare, seed, interp, flags=0):
    """Batch.project on a workspace `spare` bytes smaller than the query's."""
    import ctypes as C
    import torch
    from paper_1204_6367_amd import _abi
    L = _abi.lib()
    va, sa, p = b._structs()
    ws = b.workspace()
    out = torch.zeros(b.tally_elems, dtype=torch.float64, device="cuda")
    _abi.check(L.gdrr_mc_project_batch(va, len(b.vols), C.byref(p), sa, len(b.srcs), b._jobs_c, len(b.jobs), None, seed,
                                       (1 if interp else 0) | 2 | flags, None, out.data_ptr(), ws.data_ptr(),
                                       ws.numel() - spare, C.c_void_p(torch.cuda.current_stream().cuda_stream)))
    return out


EXTRA = 8 * 32 * 8 + 4096 * 8 + 512        # the part of the workspace that calls run without too


@pytest.mark.parametrize("interp", [True, False])
@pytest.mark.parametrize("shape, n_mat", [((1, 1, 1), 1), ((2, 3, 5), 3), ((33, 31, 35), 4), ((17, 64, 40), 9)])
def test_screened_flights_are_the_plain_ones(gpu, shape, n_mat, interp):
    """A single majorant screened by cube bounds, its chunks from eight dispensers, against
    the plain flights and one dispenser that a workspace without the extra part gets: bit for
    bit, with steep densities in one cube, zero, negative, NaN and infinite ones, materials
    beyond the table, more than eight materials (sets without a row), two volumes."""
    import torch
    rng = np.random.default_rng(3)
    names = [["air", "soft_tissue", "bone", "lung", "aluminium", "water"][k % 6] for k in range(n_mat)]
    mat = rng.integers(0, n_mat, shape).astype(np.uint8)
    dens = (10.0 ** rng.uniform(-3.0, 0.5, shape)).astype(np.float32)
    bad = dens.copy()
    bad.flat[:: 7] = rng.choice(np.array([0.0, -1.0, np.nan, np.inf], np.float32), bad.flat[:: 7].shape)
    bad_mat = mat.copy()
    bad_mat.flat[:: 11] = 250
    ph = W.Phantom(dens, mat, (200.0 / shape[2], 180.0 / shape[1], 160.0 / shape[0]), names)
    geom = W.Geometry(nu=30, nv=20, du_mm=8.0, dv_mm=8.0)
    prob = W.Problem(ph, W.physics_for(ph), W.pelvis_source(geom), geom, 1)
    vol, phys, src = gpu.upload(prob)
    vol2 = gpu.DeviceVolume(bad, bad_mat, (9.0, 8.0, 7.0) if max(shape) < 20 else ph.spacing_mm)
    jobs = [gpu.JobSpec(geom.replace(phi_rad=0.5 * k), 3001 + 17_000 * (k % 2), k, volume=k % 2) for k in range(6)]
    b = gpu.Batch([vol, vol2], phys, [src], jobs)
    got, ref = project_with(gpu, b, 0, 4, interp), project_with(gpu, b, EXTRA, 4, interp)
    assert float(ref.sum()) > 0
    assert torch.equal(got, ref)


@pytest.mark.parametrize("n_mat, tune", [(7, None), (8, None), (8, dict(block=512)), (9, dict(block=1024)), (16, None)])
def test_screened_flights_with_more_sets_than_rows(gpu, n_mat, tune):
    """Cubes of more sets of materials than the LDS has rows for (up to 247 of 8 materials, any of
    more) are screened by the row of all materials: the histories of the plain flights."""
    import torch
    rng = np.random.default_rng(n_mat)
    names = [["air", "soft_tissue", "bone", "lung", "aluminium", "water"][k % 6] for k in range(n_mat)]
    shape = (24, 26, 28)
    mat = np.zeros(shape, np.uint8)
    for _ in range(300):                                   # boxes of one material
        a = [int(rng.integers(0, s - 3)) for s in shape]
        mat[a[0]:a[0] + 4, a[1]:a[1] + 4, a[2]:a[2] + 4] = rng.integers(0, n_mat)
    dens = rng.uniform(0.01, 2.0, shape).astype(np.float32)
    ph = W.Phantom(dens, mat, (7.0, 7.0, 7.0), names)
    geom = W.Geometry(nu=30, nv=20, du_mm=8.0, dv_mm=8.0)
    prob = W.Problem(ph, W.physics_for(ph), W.pelvis_source(geom), geom, 1)
    vol, phys, src = gpu.upload(prob)
    b = gpu.Batch([vol], phys, [src], [gpu.JobSpec(geom.replace(phi_rad=0.5 * k), 30_001, k) for k in range(3)])
    ref = project_with(gpu, b, EXTRA, 4, True)
    got = b.project(seed=4, sumsq=True, tune=tune)
    assert float(ref.sum()) > 0 and torch.equal(got, ref)


@pytest.mark.parametrize("interp", [True, False])
def test_adjoint_does_not_depend_on_the_workgroup(gpu, interp):
    """The all-local adjoint at workgroups on both sides of 768 lanes, where another instantiation
    takes over: the gradient up to the order of its float64 sums (fewer than 2^23 addends of
    2^-53 each, relative to the sum of their sizes, which the largest entry bounds from below)."""
    import torch
    ph = W.ellipsoid_phantom((20, 22, 24), (12.0, 13.0, 14.0), 5, n_inner=4)
    geom = W.Geometry(nu=32, nv=24, du_mm=12.0, dv_mm=12.0)
    prob = W.Problem(ph, W.physics_for(ph), W.pelvis_source(geom), geom, 1)
    vol, phys, src = gpu.upload(prob)
    vol.local_majorants(4, 0.1, 0.05)
    b = gpu.Batch([vol], phys, [src], [gpu.JobSpec(geom, 200_003, 0)])
    maj = torch.stack([gpu.majorant(vol, phys, interp, 0.1)])
    adj = torch.ones(1, 2, 24, 32, dtype=torch.float64, device="cuda")
    ref = b.backward(adj, maj, seed=5, interp=interp)
    assert float(ref.abs().max()) > 0
    for block in (256, 768, 832, 1024):
        got = b.backward(adj, maj, seed=5, interp=interp, tune=dict(block=block))
        assert float((got - ref).abs().max()) <= 2.0**-28 * float(ref.abs().max()), block
