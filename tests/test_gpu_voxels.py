"""The pass over a volume (cell records, maxima, input checks) and the cubes' maxima at
sizes around their workgroups'."""
import numpy as np
import pytest

from paper_1204_6367_amd import workloads as W

from test_gpu_parity import compare_histories

pytestmark = pytest.mark.gpu

NAMES = ["air", "soft_tissue", "bone", "lung", "aluminium"]


@pytest.fixture(scope="module")
def gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1204_6367_amd import api
    return api


def noisy(shape, seed, n=0):
    rng = np.random.default_rng(seed)
    mat = rng.integers(0, 3, shape).astype(np.uint8)
    mat[: (shape[0] + 1) // 2] = 1
    mat.flat[-1] = 4
    dens = rng.uniform(0.2, 2.0, shape).astype(np.float32)
    ph = W.Phantom(dens, mat, (150.0 / shape[2], 140.0 / shape[1], 130.0 / shape[0]), NAMES)
    geom = W.Geometry(phi_rad=0.6, nu=24, nv=16, du_mm=12.0, dv_mm=12.0)
    spec = W.kramers_spectrum(120.0, 2.5, 2.0)
    return W.Problem(ph, W.physics_for(ph), W.Source(spec[0], spec[1], W.fluence_map(geom, spectrum=spec)), geom, n)


@pytest.mark.parametrize("interp", [True, False])
@pytest.mark.parametrize("shape", [(1, 1, 1), (1, 1, 300), (300, 1, 1), (3, 16, 15), (4, 15, 16), (5, 16, 16), (9, 31, 77)])
def test_majorant_is_the_maximum(gpu, shape, interp):
    """Exactly: per interval the largest product, in float64, of a present material's densest
    voxel (of its voxels' neighbourhoods with interpolation) and its coefficient at the
    interval's ends, rounded up to float32."""
    prob = noisy(shape, sum(shape))
    dens = prob.phantom.density
    dens.flat[:: 7] = np.array([np.nan, -1.0, 0.0], np.float32)[np.arange(dens.flat[:: 7].size) % 3]
    vol, phys, _ = gpu.upload(prob)
    d = np.where(dens >= 0, dens, 0).astype(np.float32)
    if interp:
        p = np.pad(d, 1, mode="edge")
        z, y, x = d.shape
        d = np.max([p[a:a + z, b:b + y, c:c + x] for a in range(3) for b in range(3) for c in range(3)], axis=0)
    mu = phys.mu.cpu().numpy().astype(np.float64).reshape(len(NAMES), -1, 3)
    tot = mu[..., 0] + mu[..., 1] + mu[..., 2]
    best = np.max([float(d[prob.phantom.material == m].max()) * np.maximum(tot[m, :-1], tot[m, 1:])
                   for m in np.unique(prob.phantom.material)], axis=0) * (1.0 + float(np.float32(0.125)))
    want = best.astype(np.float32)
    want = np.where(want.astype(np.float64) < best, np.nextafter(want, np.float32(np.inf)), want)
    assert np.array_equal(gpu.majorant(vol, phys, interp, 0.125).cpu().numpy(), want)


@pytest.mark.parametrize("shape, macro", [((1, 1, 1), 0), ((2, 3, 64), 0), ((5, 17, 15), 0), ((2, 3, 4), 1),
                                          ((7, 9, 8), 2), ((20, 13, 31), 7), ((30, 27, 26), 13), ((9, 70, 45), 62),
                                          ((5, 8, 140), 63), ((3, 4, 300), 256)])
def test_histories_match_oracle(gpu, shape, macro):
    """Noisy volumes whose cells mostly hold several materials: a wrong record or a cube's bound
    below its densities changes most histories."""
    import oracle
    prob = noisy(shape, sum(shape) + macro, 20_000)
    vol, phys, src = gpu.upload(prob)
    p = oracle.Problem.from_workload(prob)
    if macro:
        vol.local_majorants(macro)
        p = p.local_majorants(macro)
    g = gpu.trace(vol, phys, src, prob.geom, prob.n_photons, seed=4)
    frac, _ = compare_histories(g, oracle.mc_project(p, 4, prob.n_photons, trace=True))
    assert frac >= 0.999


@pytest.mark.parametrize("macro", [0, 5])
def test_volumes_without_photons_are_checked(gpu, macro):
    import torch
    prob = noisy((9, 8, 7), 1)
    vol, phys, src = gpu.upload(prob)
    vol.local_majorants(macro)
    bad = gpu.DeviceVolume(-prob.phantom.density, prob.phantom.material, prob.phantom.spacing_mm).local_majorants(macro)
    job = [gpu.JobSpec(prob.geom, 1000, 0)]
    b = gpu.Batch([vol, bad], phys, [src], job)
    out = b.project(seed=3)
    with pytest.raises(gpu._abi.GdrrError):
        b.input_status()
    one = gpu.Batch([vol], phys, [src], job)
    assert torch.equal(out, one.project(seed=3))
    one.input_status()


@pytest.mark.parametrize("shape", [(1000, 1, 1), (513, 1, 2), (700, 3, 4), (300, 7, 9), (257, 11, 10), (130, 10, 15)])
def test_tall_volumes(gpu, shape):
    """Few columns (4 to 176 with the cells' margin): a workgroup's lanes lie above each other too."""
    for interp in (True, False):
        test_majorant_is_the_maximum(gpu, shape, interp)
    test_histories_match_oracle(gpu, shape, 0)
