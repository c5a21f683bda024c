"""A call's tables reach the device in the arguments of a kernel or by a copy: the same tallies."""
import numpy as np
import pytest

from paper_1204_6367_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1204_6367_amd import api
    return api


# one job, around the number whose tables fill 2816 bytes (an 8-byte prefix, a record of 100 to
# 128 bytes and an 8-byte offset each, with gaps of up to 255 bytes), and many
@pytest.mark.parametrize("n_jobs", [1, 2, *range(15, 27), 90])
def test_batches_equal_single_projections(gpu, n_jobs):
    import torch
    ph = W.ellipsoid_phantom((12, 14, 16), (10.0, 9.0, 8.0), 3, n_inner=3)
    geom = W.Geometry(nu=17, nv=9, du_mm=17.0, dv_mm=25.0)
    e, w = W.kramers_spectrum(120.0, 2.5, 2.0)
    prob = W.Problem(ph, W.physics_for(ph), W.Source(e, w, np.ones((9, 17), np.float32)), geom, 0)
    vol, phys, src = gpu.upload(prob)
    jobs = [gpu.JobSpec(geom.replace(phi_rad=0.3 * k), 100 + 37 * k, k) for k in range(n_jobs)]
    b = gpu.Batch([vol], phys, [src], jobs)
    tallies = b.project(seed=5).reshape(n_jobs, -1)
    images = b.primary()
    for k in {0, n_jobs // 2, n_jobs - 1}:
        one = gpu.Batch([vol], phys, [src], [jobs[k]])
        assert torch.equal(tallies[k], one.project(seed=5).reshape(-1))
        assert torch.equal(images[k], one.primary()[0])
