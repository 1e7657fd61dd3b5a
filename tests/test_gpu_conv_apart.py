"""FP32 problems of 5 and 6 layers of up to 256 rows, which both the in-place
convolution (k_convz) and k_conv with its separate output can take: the same
bits by either route (alone, k_conv; beside a problem whose spectra fill most of the
last-level cache, in place), and the allocation-free evaluation takes them in
place where the separate output would not fit its scratch."""
import pytest
import torch

from paper_1804_07135_amd import ssm

pytestmark = pytest.mark.gpu


def _spins(p, seed):
    s = torch.randn((p["K"], 3, p["nz"], p["ny"], p["nx"]), device="cuda",
                    generator=torch.Generator(device="cuda").manual_seed(seed))
    return s / s.norm(dim=1, keepdim=True)


@pytest.mark.parametrize("ny", [193, 251, 256])
def test_same_bits_by_either_route(ny):
    p = dict(nx=9, ny=ny, nz=5, K=3, J=0.9, d=0.35, ku=0.21, D=0.4)
    s = _spins(p, ny)
    h = ssm.StringMethod(p, ssm.SSM_FP32_MIXED).eval(s)[1]
    # 257 kx of 15 lines of 250 values, 18 images: 132 MiB of spectra
    big = dict(p, nx=250, ny=250, K=18)
    hb = ssm.StringMethod([p, big], ssm.SSM_FP32_MIXED).eval(torch.cat([s.reshape(-1), _spins(big, 1).reshape(-1)]))[1]
    assert torch.equal(hb.reshape(-1)[:h.numel()], h.reshape(-1))


@pytest.mark.parametrize("nz", [5, 6])
def test_noalloc_in_place_where_the_scratch_asks_for_it(nz):
    # X alone about 40 (48) MB, with a separate output over 64 MiB
    p = dict(nx=32, ny=250, nz=nz, K=40, J=0.9, d=0.35, ku=0.21, D=0.02)
    s = _spins(p, nz)
    E, h, T = ssm.StringMethod(p, ssm.SSM_FP32_MIXED).eval(s)
    En, hn, Tn = torch.empty_like(E), torch.empty_like(s), torch.empty_like(T)
    ssm.ssm_eval_noalloc([p], ssm.SSM_FP32_MIXED, s, hn, En, Tn)
    torch.cuda.synchronize()
    assert torch.equal(hn.reshape(-1), h.reshape(-1)) and torch.equal(En, E) and torch.equal(Tn, T)
