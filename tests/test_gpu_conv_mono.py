"""The monolayer convolution (k_conv1) at the edges of every y length it is
built for: the shortest line that takes the length, one short of it, and the
whole length, odd and even; image counts that leave its image groups ragged.
Fields against the oracle at 1e-10 (FP64) and 1e-5 (FP32-mixed), and bitwise
the same whatever number of images a workgroup takes (forced through a tile
cache)."""
import numpy as np
import pytest
import torch

from paper_1804_07135_amd import inputs, ssm

pytestmark = pytest.mark.gpu

TOL = {ssm.SSM_FP64: 1e-10, ssm.SSM_FP32_MIXED: 1e-5}


@pytest.mark.parametrize("precision", [ssm.SSM_FP64, ssm.SSM_FP32_MIXED])
@pytest.mark.parametrize("ny,K", [(17, 18), (32, 2), (33, 11), (47, 3), (48, 2), (49, 12), (64, 2), (65, 11),
                                  (95, 3), (96, 2), (97, 9), (128, 3), (129, 6), (191, 2), (192, 3), (193, 3),
                                  (255, 2), (256, 3)])
def test_monolayer_lengths_vs_oracle(oracle, tmp_path, precision, ny, K):
    p = dict(nx=3, ny=ny, nz=1, K=K, J=0.9, d=0.35, ku=0.21, D=0.4)
    s = inputs.random_unit_spins((K, 3, 1, ny, 3), seed=ny)
    if precision == ssm.SSM_FP32_MIXED:
        s = s.astype(np.float32).astype(np.float64)
    sm = ssm.StringMethod(p, precision)
    h = sm.eval(s)[1]
    for k in (0, K // 2, K - 1):
        ho = oracle.field(s[k], p["J"], p["d"], p["ku"], p["D"])
        assert np.abs(h[k].cpu().numpy() - ho).max() < TOL[precision] * np.abs(ho).max(), k
    dev = torch.cuda.get_device_properties(0).gcnArchName.replace(" ", "_")
    for g in (1, 2, 64):
        cache = tmp_path / f"tiles{g}"
        cache.write_text(f"{dev} {precision} 3x{ny}x1 {K} 8 4 {g}\n")
        sm.set_string(s)
        sm.autotune(str(cache))
        assert torch.equal(sm.eval(s)[1], h), g
