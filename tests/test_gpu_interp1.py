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


@pytest.mark.parametrize("precision", [ssm.SSM_FP64, ssm.SSM_FP32_MIXED])
@pytest.mark.parametrize("climb", [False, True])
@pytest.mark.parametrize("kind", ["spline", "two", "repeat", "still"])
def test_spline_pass_takes_degenerate_splines(precision, climb, kind):
    """The one-pass spline step of problems with few images (k_interp_splw)
    takes a degenerate spline's linear step too: bitwise what k_interp gives
    such a problem in a batch with one of more images (two images, two equal
    neighbours, no arc length at all)."""
    K = 2 if kind == "two" else 6
    p = dict(nx=9, ny=7, nz=1, K=K, J=0.9, d=0.35, ku=0.21, D=0.02)
    s = inputs.random_unit_spins((K, 3, 1, 7, 9), seed=3)
    if kind == "repeat":
        s[3] = s[2]
    if kind == "still":
        s[:] = s[:1]
    long = dict(p, nx=3, ny=2, K=40)
    sl = inputs.random_unit_spins((40, 3, 1, 2, 3), seed=1)
    one, two = ssm.StringMethod(p, precision), ssm.StringMethod([p, long], precision)
    out = []
    for sm, x in ((one, s.ravel()), (two, np.concatenate([s.ravel(), sl.ravel()]))):
        sm.set_reparam(ssm.SSM_INTERP_SPLINE, climb)
        sm.set_string(x.reshape(s.shape) if sm is one else x)
        assert sm.iterate(3, 0.1).tolist()[0] == 3
        out.append(sm.get_string().reshape(-1)[:s.size])
    assert torch.equal(out[0], out[1])


@pytest.mark.parametrize("precision,K", [(ssm.SSM_FP64, 3), (ssm.SSM_FP64, 5), (ssm.SSM_FP64, 16),
                                         (ssm.SSM_FP32_MIXED, 8), (ssm.SSM_FP32_MIXED, 9), (ssm.SSM_FP32_MIXED, 30)])
@pytest.mark.parametrize("nx,ny", [(20, 18), (17, 31), (16, 31)])
def test_degenerate_splines_in_rounds_of_images(precision, K, nx, ny):
    """The same at image counts on both sides of the pass's rounds and on
    lattices of several workgroups, the last one ragged, whose sites k_interp
    takes four (two in FP64) or one to a thread; the degenerate problem second in its
    batch, behind one whose spline is not."""
    p = dict(nx=nx, ny=ny, nz=1, K=K, J=0.9, d=0.35, ku=0.21, D=0.02)
    s = inputs.random_unit_spins((K, 3, 1, ny, nx), seed=K)
    s[1] = s[0]  # two equal neighbours
    first = dict(p, nx=11, ny=5, K=7)
    sf = inputs.random_unit_spins((7, 3, 1, 5, 11), seed=2)
    long = dict(p, nx=3, ny=2, K=40)
    sl = inputs.random_unit_spins((40, 3, 1, 2, 3), seed=1)
    out = []
    for probs, x in (([first, p], [sf, s]), ([first, p, long], [sf, s, sl])):
        sm = ssm.StringMethod(probs, precision)
        sm.set_reparam(ssm.SSM_INTERP_SPLINE, False)
        sm.set_string(np.concatenate([v.ravel() for v in x]))
        sm.iterate(1, 0.0)  # (no step: the spline stays degenerate)
        out.append(sm.get_string().reshape(-1)[:sf.size + s.size])
    assert torch.equal(out[0], out[1])
