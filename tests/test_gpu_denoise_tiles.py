"""How an image is cut into regions does not show in the denoised result."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1204_6367_amd import api
    return api


def images(seed, n, nv, nu):
    rng = np.random.default_rng(seed)
    y, x = np.mgrid[0:nv, 0:nu]
    a = rng.poisson(90.0 + 60.0 * np.sin(x / 7.0) * np.cos(y / 9.0), (n, nv, nu)).astype(np.float64)
    a[:, : 3, : 5] = 0.0
    a[:, nv // 2, nu // 2] = 0.0
    return a


def sweeps_f64(shat, beta, omega, iters, floor):
    s = np.maximum(shat, floor)
    for _ in range(iters):
        p = np.pad(s, ((1, 1), (1, 1)), mode="edge")
        data = np.where(shat == 0.0, 1.0, 1.0 - shat / s)
        s = np.maximum((1 - omega) * s + omega / 4 * (p[:-2, 1:-1] + p[2:, 1:-1] + p[1:-1, :-2] + p[1:-1, 2:] - data / beta), floor)
    return s


# heights and widths at, below and above the regions' (56, 80, 96 and 112 rows; 64 and 128 columns)
@pytest.mark.parametrize("nv, nu", [(1, 1), (2, 65), (55, 64), (56, 64), (57, 63), (80, 129), (81, 128), (96, 127),
                                    (97, 64), (112, 65), (113, 193), (240, 256), (192, 128), (384, 64)])
@pytest.mark.parametrize("iters", [1, 25, 50])
def test_few_and_many_images(gpu, nv, nu, iters):
    """One image, few and more than the chip holds at once take regions of different
    sizes, halos and wavefronts, or whole images per workgroup: the same bits.  The first
    agrees with float64 sweeps to the float32 rounding of each sweep: (iters + 2) 2^-22 of
    the image's scale."""
    import torch
    a = images(nv * 7 + nu + iters, 9, nv, nu)
    x = torch.tensor(a, device="cuda")
    one = [gpu.denoise(x[k], 0.05, iters, s_floor=1e-3) for k in (0, 8)]
    for n in (9, 300, 1200):
        many = gpu.denoise(x.repeat((n + 8) // 9, 1, 1)[:n].contiguous(), 0.05, iters, s_floor=1e-3)
        assert torch.equal(many[0], one[0])
        assert torch.equal(many[(n - 9) // 9 * 9 + 8], one[1])
    ref = sweeps_f64(a[0], 0.05, 0.8, iters, 1e-3)
    assert np.abs(one[0].cpu().numpy() - ref).max() <= (iters + 2) * 2.0**-22 * np.abs(ref).max()


def test_floor_below_the_normal_numbers_and_a_workspace_without_the_third_buffer(gpu):
    """Where Shat = 0 the data term is 1 by a comparison only if an iterate may be too small
    for the reciprocal; Shat is read as doubles by every pass if the workspace has no room
    for its float32 copy.  Neither shows in the result."""
    import torch
    from paper_1204_6367_amd import _abi
    L = _abi.lib()
    x = torch.tensor(images(3, 2, 150, 200), device="cuda")
    ref = gpu.denoise(x, 0.05, 60, s_floor=1.2e-38)
    low = gpu.denoise(x, 0.05, 60, s_floor=1e-39)
    held = ref == float(np.float32(1.2e-38))               # pixels at the floor itself
    assert torch.equal(low[~held], ref[~held]) and torch.all(low[held] == float(np.float32(1e-39)))
    ws = torch.empty(2 * ((2 * 150 * 200 * 4 + 255) // 256 * 256) + 256, dtype=torch.uint8, device="cuda")
    out = torch.empty_like(ref)
    _abi.check(L.gdrr_denoise(x.data_ptr(), 0, 2, 150, 200, 0.05, 0.8, 60, 1.2e-38, out.data_ptr(), ws.data_ptr(),
                              ws.numel(), torch.cuda.current_stream().cuda_stream))
    assert torch.equal(out, ref)
