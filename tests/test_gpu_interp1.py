"""Step 2 with the reduction inside the interpolation's launch (k_interp1, every
problem with few images and partials, linear, no climbing image): bitwise the
results of the two launches that serve a batch in which one problem has more
images than that, at the edges of the image count and of the sites per chunk."""
import numpy as np
import pytest
import torch

from paper_1804_07135_amd import inputs, ssm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", [ssm.SSM_FP64, ssm.SSM_FP32_MIXED])
@pytest.mark.parametrize("nx,ny,nz,K,still", [(2, 3, 1, 2, False), (5, 7, 1, 3, False), (16, 16, 1, 63, False),
                                              (17, 31, 1, 64, False), (32, 33, 2, 10, False), (16, 64, 1, 5, True),
                                              (64, 65, 1, 64, False)])
def test_same_as_two_launches(precision, nx, ny, nz, K, still):
    p = dict(nx=nx, ny=ny, nz=nz, K=K, J=0.9, d=0.35, ku=0.21, D=0.02)
    s = inputs.random_unit_spins((K, 3, nz, ny, nx), seed=K)
    if still:
        s = np.broadcast_to(s[:1], s.shape).copy()  # no arc length: every image is copied
    long = dict(nx=3, ny=2, nz=nz, K=65, J=0.9, d=0.35, ku=0.21, D=0.02)
    sl = inputs.random_unit_spins((65, 3, nz, 2, 3), seed=1)
    one, two = ssm.StringMethod([p, p], precision), ssm.StringMethod([p, long, p], precision)
    one.set_string(np.concatenate([s.ravel(), s[::-1].ravel()]))
    two.set_string(np.concatenate([s.ravel(), sl.ravel(), s[::-1].ravel()]))
    it1, it2 = one.iterate(3, 0.1), two.iterate(3, 0.1)
    assert it1.tolist() == [3, 3] and it2.tolist() == [3, 3, 3]
    a, b = one.get_string().reshape(-1), two.get_string().reshape(-1)
    n = s.size
    assert torch.equal(a[:n], b[:n]) and torch.equal(a[n:], b[n + sl.size:])
    e, f = one.energies(), two.energies()
    assert torch.equal(e[:K], f[:K]) and torch.equal(e[K:], f[K + 65:])
