"""The inverse x transform in two register steps (xinv_two_step) at the edges
of every length it serves, odd and even row counts, and row tiles from two
rows to beyond what it takes (where the kernel goes one component at a time):
fields against the oracle at 1e-10 (FP64) and 1e-5 (FP32-mixed), and bitwise
the same for every tile (rows are transformed in pairs that no tile splits)."""
import numpy as np
import pytest
import torch

from paper_1804_07135_amd import inputs, ssm

pytestmark = pytest.mark.gpu

TOL = {ssm.SSM_FP64: 1e-10, ssm.SSM_FP32_MIXED: 1e-5}


@pytest.mark.parametrize("precision", [ssm.SSM_FP64, ssm.SSM_FP32_MIXED])
@pytest.mark.parametrize("nx,ny,nz", [(17, 6, 2), (32, 5, 1), (33, 7, 1), (48, 2, 3), (49, 9, 1), (64, 4, 1), (65, 5, 2),
                                      (95, 6, 1), (96, 3, 1), (97, 8, 1), (128, 5, 1), (129, 1, 1), (192, 4, 1),
                                      (193, 3, 1), (255, 2, 2), (256, 5, 1)])
def test_inverse_x_lengths_and_tiles_vs_oracle(oracle, tmp_path, precision, nx, ny, nz):
    p = dict(nx=nx, ny=ny, nz=nz, K=2, J=0.9, d=0.35, ku=0.21, D=0.4)
    s = inputs.random_unit_spins((2, 3, nz, ny, nx), seed=nx)
    if precision == ssm.SSM_FP32_MIXED:
        s = s.astype(np.float32).astype(np.float64)
    sm = ssm.StringMethod(p, precision)
    h = sm.eval(s)[1]
    for k in range(2):
        ho = oracle.field(s[k], p["J"], p["d"], p["ku"], p["D"])
        assert np.abs(h[k].cpu().numpy() - ho).max() < TOL[precision] * np.abs(ho).max(), k
    dev = torch.cuda.get_device_properties(0).gcnArchName.replace(" ", "_")
    sm.set_string(s)
    for rows in (2, 4, 8, 16, 32, 64, 128):
        if 3 * rows * nx * s.itemsize > 60000:
            break  # tiles beyond this may not fit in LDS at all
        cache = tmp_path / f"tiles{rows}"
        cache.write_text(f"{dev} {precision} {nx}x{ny}x{nz} 2 8 {rows} 1\n")
        sm.autotune(str(cache))
        assert torch.equal(sm.eval(s)[1], h), rows


@pytest.mark.parametrize("precision", [ssm.SSM_FP64, ssm.SSM_FP32_MIXED])
@pytest.mark.parametrize("nx,ny,nz", [(1, 3, 1), (31, 33, 1), (33, 64, 2), (63, 31, 3), (64, 65, 1)])
def test_wide_workgroups(oracle, precision, nx, ny, nz):
    """The shortest power-of-two lengths (workgroups of kXinvWide threads):
    field and energy against the oracle, and bitwise the same in a batch with
    problems of the other kinds."""
    p = dict(nx=nx, ny=ny, nz=nz, K=3, J=0.9, d=0.35, ku=0.21, D=0.4)
    s = inputs.random_unit_spins((3, 3, nz, ny, nx), seed=nx + ny)
    if precision == ssm.SSM_FP32_MIXED:
        s = s.astype(np.float32).astype(np.float64)
    E, h = ssm.StringMethod(p, precision).eval(s)[:2]
    for k in range(3):
        ho = oracle.field(s[k], p["J"], p["d"], p["ku"], p["D"])
        assert np.abs(h[k].cpu().numpy() - ho).max() < TOL[precision] * np.abs(ho).max(), k
        scale = 0.5 * np.abs(s[k] * ho).sum()
        assert abs(E[k].item() + 0.5 * (s[k] * ho).sum()) < TOL[precision] * scale, k
    others = [dict(p, nx=45, K=2), dict(p, nx=100, K=2)]
    so = [inputs.random_unit_spins((2, 3, nz, ny, q["nx"]), seed=5) for q in others]
    batch = ssm.StringMethod([others[0], p, others[1]], precision)
    Eb, hb = batch.eval(np.concatenate([so[0].ravel(), s.ravel(), so[1].ravel()]))[:2]
    assert torch.equal(Eb[2:5], E)
    assert torch.equal(hb.reshape(-1)[so[0].size:so[0].size + s.size], h.reshape(-1))


@pytest.mark.parametrize("precision,nx", [(ssm.SSM_FP64, 17), (ssm.SSM_FP64, 31), (ssm.SSM_FP64, 32),
                                          (ssm.SSM_FP32_MIXED, 17), (ssm.SSM_FP32_MIXED, 32), (ssm.SSM_FP32_MIXED, 49),
                                          (ssm.SSM_FP32_MIXED, 63), (ssm.SSM_FP32_MIXED, 64)])
@pytest.mark.parametrize("ny,nz", [(33, 1), (1, 2), (7, 3), (64, 2)])
def test_wide_workgroup_lengths(oracle, precision, nx, ny, nz):
    """Every length that takes workgroups of kXinvWide threads (half lengths 32
    and, FP32, 64) at its shortest and longest rows, odd and even row counts
    and several layers: field and energy against the oracle, and bitwise the
    same beside problems of the other kinds (the rest of test_wide_workgroups'
    rows take 256 threads)."""
    p = dict(nx=nx, ny=ny, nz=nz, K=2, J=0.9, d=0.35, ku=0.21, D=0.4)
    s = inputs.random_unit_spins((2, 3, nz, ny, nx), seed=nx + ny)
    if precision == ssm.SSM_FP32_MIXED:
        s = s.astype(np.float32).astype(np.float64)
    E, h = ssm.StringMethod(p, precision).eval(s)[:2]
    for k in range(2):
        ho = oracle.field(s[k], p["J"], p["d"], p["ku"], p["D"])
        assert np.abs(h[k].cpu().numpy() - ho).max() < TOL[precision] * np.abs(ho).max(), k
        scale = 0.5 * np.abs(s[k] * ho).sum()
        assert abs(E[k].item() + 0.5 * (s[k] * ho).sum()) < TOL[precision] * scale, k
    others = [dict(p, nx=40), dict(p, nx=110)]
    so = [inputs.random_unit_spins((2, 3, nz, ny, q["nx"]), seed=5) for q in others]
    batch = ssm.StringMethod([others[0], p, others[1]], precision)
    Eb, hb = batch.eval(np.concatenate([so[0].ravel(), s.ravel(), so[1].ravel()]))[:2]
    assert torch.equal(Eb[2:4], E)
    assert torch.equal(hb.reshape(-1)[so[0].size:so[0].size + s.size], h.reshape(-1))
