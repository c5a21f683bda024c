"""Source tables at the sizes where their preparation changes: photons leave in the directions
and with the energies that the oracle's tables give them."""
import numpy as np
import pytest

from paper_1204_6367_amd import workloads as W

from test_gpu_parity import compare_histories
from test_gpu_raytrace import check_image

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1204_6367_amd import api
    return api


# up to 2048 pixels in one workgroup, above in 16; segments of 1, 2, 3, 64, 65 and 68 pixels;
# up to 4096 rows of a joint source a workgroup each, above in turns
@pytest.mark.parametrize("nu, nv, joint", [(1, 1, False), (3, 5, True), (32, 64, False), (2049, 1, False), (3, 683, True),
                                           (83, 37, True), (5000, 1, True), (256, 256, False), (257, 256, False), (67, 1031, False)])
def test_photons_start_as_in_the_oracle(gpu, nu, nv, joint):
    import oracle
    rng = np.random.default_rng(nu + nv)
    ph = W.ellipsoid_phantom((12, 14, 16), (10.0, 9.0, 8.0), 3, n_inner=3)
    geom = W.Geometry(phi_rad=0.6, nu=nu, nv=nv, du_mm=300.0 / nu, dv_mm=250.0 / nv)
    e, w = W.kramers_spectrum(120.0, 2.5, 2.0)
    flu = rng.uniform(0.0, 1.0, (nv, nu)).astype(np.float32) ** 8
    flu.flat[rng.integers(0, flu.size, flu.size // 3)] = 0.0
    flu.flat[-1] = 1.0
    if joint:
        w = (w * rng.uniform(0.0, 1.0, (nu, len(w)))).astype(np.float32)
        w[:, ::3] = 0.0
    prob = W.Problem(ph, W.physics_for(ph), W.Source(e, w, flu), geom, 30_000)
    vol, phys, src = gpu.upload(prob)
    g = gpu.trace(vol, phys, src, geom, prob.n_photons, seed=9)
    o = oracle.Problem.from_workload(prob)
    frac, _ = compare_histories(g, oracle.mc_project(o, 9, prob.n_photons, trace=True))
    assert frac >= 0.999
    if joint:
        check_image(gpu.primary(vol, phys, src, geom).cpu().numpy(), oracle.primary_raytrace(o), "joint")


@pytest.mark.parametrize("nu, nv", [(5, 4), (100, 30)])
def test_bad_weights_anywhere_are_reported(gpu, nu, nv):
    ph = W.ellipsoid_phantom((12, 14, 16), (10.0, 9.0, 8.0), 3, n_inner=3)
    geom = W.Geometry(nu=nu, nv=nv, du_mm=300.0 / nu, dv_mm=250.0 / nv)
    e, w = W.kramers_spectrum(120.0, 2.5, 2.0)
    for at, value in ((0, np.nan), (nu * nv // 2, -1.0), (nu * nv - 1, np.inf), (None, 0.0)):
        flu = np.ones((nv, nu), np.float32)
        if at is None:
            flu[:] = 0.0
        else:
            flu.flat[at] = value
        prob = W.Problem(ph, W.physics_for(ph), W.Source(e, w, flu), geom, 100)
        vol, phys, src = gpu.upload(prob)
        b = gpu.Batch([vol], phys, [src], [gpu.JobSpec(geom, 100, 0)])
        b.project(seed=1)
        with pytest.raises(gpu._abi.GdrrError) as err:
            b.input_status()
        assert "weights" in str(err.value)
        b.primary()
        with pytest.raises(gpu._abi.GdrrError):
            gpu.input_status(b._rt_ws)
