"""The FP32 transform from planes where it leaves its tiles for the general path
and comes back to them: both ends of that range of sites, and the dense plane
strides near a multiple of 4 MiB within it, dense, padded and with an odd pitch;
bit for bit against torch's permutation, with nothing written around the lattice."""

import pytest
import torch

from _gpu import dev, say

pytestmark = pytest.mark.gpu

NEAR = 16384     # sites of 8 bytes in 128 KiB
SITES = [500000, 500016, 524288 - NEAR, 524288, 524288 + NEAR, 700000, 2 ** 20 - NEAR + 16, 2 ** 20, 2 ** 20 + NEAR,
         1449984, 1450000, 1450016]


@pytest.mark.parametrize("sites", SITES)
def test_from_planes(sites):
    from paper_2103_00571_amd import abi

    gen = torch.Generator(device="cuda")
    gen.manual_seed(sites)
    for pitch in (sites, (sites + 63) // 64 * 64 + 128, sites + 1):
        say("from planes sites=%d pitch=%d" % (sites, pitch))
        planes = torch.full((36, pitch), float("nan"), dtype=torch.complex64, device=dev())
        planes[:, :sites] = torch.randn((36, sites), dtype=torch.complex64, device=dev(), generator=gen)
        back = torch.full((sites + 2, 36), float("nan"), dtype=torch.complex64, device=dev())
        assert abi.su3_soa_to_aos_pitched(planes.data_ptr(), back[1:].data_ptr(), sites, pitch, abi.SU3_F32,
                                          torch.cuda.current_stream().cuda_stream) == 0
        torch.cuda.synchronize()
        assert torch.equal(back[1:sites + 1], planes[:, :sites].t())
        assert bool(torch.isnan(back[0].real).all()) and bool(torch.isnan(back[-1].real).all())
