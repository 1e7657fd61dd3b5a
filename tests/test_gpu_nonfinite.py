"""A spin that is not finite: the dipolar field couples every component of
every site to it (a monolayer's zero tensor elements times NaN or infinity
among them), so it shows in the whole field of its image, as in the oracle's
direct sum, at every kind of y length; other images keep their bits."""
import numpy as np
import pytest
import torch

from paper_1804_07135_amd import inputs, ssm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", [ssm.SSM_FP64, ssm.SSM_FP32_MIXED])
@pytest.mark.parametrize("ny,nz", [(12, 1), (24, 1), (48, 1), (57, 1), (96, 1), (120, 1), (192, 1), (250, 1), (300, 1),
                                   (24, 2), (192, 4)])
def test_whole_field_shows_a_nonfinite_spin(oracle, precision, ny, nz):
    nx, K = 5, 12  # more images than some workgroups take
    p = dict(nx=nx, ny=ny, nz=nz, K=K, J=0.9, d=0.35, ku=0.21, D=0.4)
    s = inputs.random_unit_spins((K, 3, nz, ny, nx), seed=ny)
    sm = ssm.StringMethod(p, precision)
    E, h = sm.eval(s)[:2]
    for value, c, k in ((np.nan, 0, 0), (np.nan, 2, 7), (np.inf, 1, 11), (-np.inf, 2, 4)):
        b = s.copy()
        b[k, c, 0, ny // 2, 1] = value
        with np.errstate(invalid="ignore"):
            ho = oracle.field(b[k], p["J"], p["d"], p["ku"], p["D"])
        Eb, hb = sm.eval(b)[:2]
        assert not torch.isfinite(hb[k].cpu()[torch.as_tensor(~np.isfinite(ho))]).any(), (value, c)
        assert not torch.isfinite(Eb[k])
        rest = [i for i in range(K) if i != k]
        assert torch.equal(hb[rest], h[rest]) and torch.equal(Eb[rest], E[rest]), (value, c)
