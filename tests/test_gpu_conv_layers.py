"""The in-place convolution of several layers (k_convz) at the edges of its
y lengths, for layer counts at both ends of a padded count and on both sides of
the one where a slice no longer fits in LDS with both halves (k_conv then):
fields against the oracle at 1e-10 (FP64) and 1e-5 (FP32-mixed), and bitwise
the same whatever number of images a workgroup takes."""
import numpy as np
import pytest
import torch

from paper_1804_07135_amd import inputs, ssm

pytestmark = pytest.mark.gpu

TOL = {ssm.SSM_FP64: 1e-10, ssm.SSM_FP32_MIXED: 1e-5}


@pytest.mark.parametrize("precision", [ssm.SSM_FP64, ssm.SSM_FP32_MIXED])
@pytest.mark.parametrize("ny,nz,K", [(17, 2, 5), (32, 8, 2), (33, 3, 7), (48, 4, 2), (49, 5, 3), (64, 2, 9), (65, 7, 2),
                                     (96, 4, 3), (96, 8, 2), (97, 3, 3), (128, 4, 2), (128, 5, 2), (128, 7, 2),
                                     (129, 2, 3), (191, 3, 2), (192, 4, 2), (192, 8, 2), (193, 2, 2), (255, 3, 2),
                                     (256, 4, 2), (256, 5, 2), (250, 6, 2), (256, 7, 2)])
def test_layered_lengths_vs_oracle(oracle, tmp_path, precision, ny, nz, K):
    p = dict(nx=2, ny=ny, nz=nz, K=K, J=0.9, d=0.35, ku=0.21, D=0.4)
    s = inputs.random_unit_spins((K, 3, nz, ny, 2), seed=ny + nz)
    if precision == ssm.SSM_FP32_MIXED:
        s = s.astype(np.float32).astype(np.float64)
    sm = ssm.StringMethod(p, precision)
    h = sm.eval(s)[1]
    for k in (0, K - 1):
        ho = oracle.field(s[k], p["J"], p["d"], p["ku"], p["D"])
        assert np.abs(h[k].cpu().numpy() - ho).max() < TOL[precision] * np.abs(ho).max(), k
    dev = torch.cuda.get_device_properties(0).gcnArchName.replace(" ", "_")
    sm.set_string(s)
    for g in (1, 2, 3):
        cache = tmp_path / f"tiles{g}"
        cache.write_text(f"{dev} {precision} 2x{ny}x{nz} {K} 8 4 {g}\n")
        try:
            sm.autotune(str(cache))
        except ssm.SSMError as e:  # more slices than fit (the half-by-half kernel takes what it is given)
            assert e.status == ssm.SSM_EUNSUPPORTED
            continue
        assert torch.equal(sm.eval(s)[1], h), g


@pytest.mark.parametrize("ny,nz", [(129, 4), (161, 4), (193, 3), (193, 4), (241, 4), (256, 3)])
def test_halves_kernel_edges(oracle, ny, nz):
    """FP64, 3 and 4 layers at the y lengths of the half-by-half kernel of one
    slice per workgroup (k_convh): shortest, ragged and longest lines, an odd
    number of x columns and of images, alone and beside another problem."""
    p = dict(nx=3, ny=ny, nz=nz, K=3, J=0.9, d=0.35, ku=0.21, D=0.4)
    s = inputs.random_unit_spins((3, 3, nz, ny, 3), seed=ny * nz)
    h = ssm.StringMethod(p, ssm.SSM_FP64).eval(s)[1]
    for k in range(3):
        ho = oracle.field(s[k], p["J"], p["d"], p["ku"], p["D"])
        assert np.abs(h[k].cpu().numpy() - ho).max() < 1e-10 * np.abs(ho).max(), k
    q = dict(p, ny=200, K=2)
    s2 = inputs.random_unit_spins((2, 3, nz, 200, 3), seed=1)
    both = ssm.StringMethod([q, p], ssm.SSM_FP64)
    hb = both.eval(torch.cat([torch.as_tensor(s2).reshape(-1), torch.as_tensor(s).reshape(-1)]))[1]
    assert torch.equal(hb.reshape(-1)[-h.numel():].cpu(), h.reshape(-1).cpu())


@pytest.mark.parametrize("ny", [130, 192, 194, 256])
def test_halves_kernel_four_layers(oracle, ny):
    """FP64, 4 layers, the one layer count that k_convh serves (3 layers of these
    lengths fit in k_convz): the shortest even and the whole lines of both its
    lengths, more images than XCDs, alone and beside a problem of 3 layers."""
    K = 9
    p = dict(nx=2, ny=ny, nz=4, K=K, J=0.9, d=0.35, ku=0.21, D=0.4)
    s = inputs.random_unit_spins((K, 3, 4, ny, 2), seed=ny)
    h = ssm.StringMethod(p, ssm.SSM_FP64).eval(s)[1]
    for k in (0, K - 1):
        ho = oracle.field(s[k], p["J"], p["d"], p["ku"], p["D"])
        assert np.abs(h[k].cpu().numpy() - ho).max() < 1e-10 * np.abs(ho).max(), k
    q = dict(p, nz=3, K=2)
    s2 = inputs.random_unit_spins((2, 3, 3, ny, 2), seed=1)
    h2 = ssm.StringMethod(q, ssm.SSM_FP64).eval(s2)[1]
    both = ssm.StringMethod([q, p], ssm.SSM_FP64)
    hb = both.eval(torch.cat([torch.as_tensor(s2).reshape(-1), torch.as_tensor(s).reshape(-1)]))[1].reshape(-1)
    assert torch.equal(hb[:h2.numel()], h2.reshape(-1)) and torch.equal(hb[h2.numel():], h.reshape(-1))
