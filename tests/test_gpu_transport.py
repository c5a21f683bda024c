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


@pytest.mark.parametrize("macro", [0, 4])
@pytest.mark.parametrize("n_e", [299, 1023])
def test_tallies_do_not_depend_on_started_photons_kept(gpu, macro, n_e):
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
    ref = b.project(seed=3, tune=dict(block=64, chunk=64))
    assert float(ref.sum()) > 0
    for t in (None, dict(block=512, defer=1), dict(block=1024, defer=8, chunk=128), dict(block=1024, blocks_per_cu=1)):
        print("shape", t, flush=True)
        assert torch.equal(b.project(seed=3, tune=t), ref), t
