"""The layout transforms at the sizes, pitches and base addresses where their
tile, halo and 16-byte paths begin and end: bit for bit against torch's
permutation, with nothing written outside the lattice part of the planes."""

import pytest
import torch

from _gpu import dev, say

pytestmark = pytest.mark.gpu

SITES = [15, 4095, 49152, 49153, 49168, 65536, 65537, 65600, 131072, 131073, 131080, 131088,
         196607, 196608, 196609, 196640, 200003, 524285]


def _pitches(n):
    up = (n + 127) // 128 * 128
    return sorted({n, n + 1, n + 2, up, up + 16, up + 65})


@pytest.mark.parametrize("offset", [0, 16, 64])    # bytes of the planes past a 128-byte line
@pytest.mark.parametrize("dtype", [torch.complex128, torch.complex64])
@pytest.mark.parametrize("sites", SITES)
def test_transforms_at_the_edges(sites, dtype, offset):
    from paper_2103_00571_amd import abi

    form, es = (abi.SU3_F64, 16) if dtype == torch.complex128 else (abi.SU3_F32, 8)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(sites)
    x = torch.randn((sites, 36), dtype=dtype, device=dev(), generator=gen)
    want = x.t().contiguous()
    stream = torch.cuda.current_stream().cuda_stream
    for pitch in _pitches(sites):
        say("transpose sites=%d pitch=%d %s offset=%d" % (sites, pitch, dtype, offset))
        lead = offset // es
        whole = torch.full((lead + 36 * pitch + 64,), float("nan"), dtype=dtype, device=dev())
        planes = whole[lead:lead + 36 * pitch].view(36, pitch)
        assert planes.data_ptr() % 128 == offset
        assert abi.su3_aos_to_soa_pitched(x.data_ptr(), planes.data_ptr(), sites, pitch, form, stream) == 0
        torch.cuda.synchronize()
        assert torch.equal(planes[:, :sites], want)
        # nothing before, between or after the planes' lattice parts was touched
        kept = torch.isnan(whole.real)
        assert int(kept.sum()) == whole.numel() - 36 * sites
        back = torch.full((sites + 2, 36), float("nan"), dtype=dtype, device=dev())
        assert abi.su3_soa_to_aos_pitched(planes.data_ptr(), back[1:].data_ptr(),
                                          sites, pitch, form, stream) == 0
        torch.cuda.synchronize()
        assert torch.equal(back[1:sites + 1], x)
        assert bool(torch.isnan(back[0].real).all()) and bool(torch.isnan(back[-1].real).all())


# Both sides of the sizes where the write-through forms begin and end, and a
# tail of tiles shorter than one group of the tile order.
@pytest.mark.parametrize("dtype", [torch.complex128, torch.complex64])
@pytest.mark.parametrize("sites", [65552, 131104, 200000, 262144, 262160, 400000, 400016, 525328,
                                   500000, 500016, 1041664, 1041680, 1100000, 1100032])
def test_grouped_and_write_through_tiles(sites, dtype):
    test_transforms_at_the_edges(sites, dtype, 0)


# Planes that span more than the 4 GiB that a 32-bit offset reaches.
@pytest.mark.parametrize("dtype", [torch.complex128, torch.complex64])
@pytest.mark.parametrize("pitch", [7 << 20, (7 << 20) + 16, (15 << 20) + 16])
def test_long_plane_strides(pitch, dtype):
    from paper_2103_00571_amd import abi

    form, sites = (abi.SU3_F64 if dtype == torch.complex128 else abi.SU3_F32), 140000
    if pitch > 15 << 20:
        sites = 1100048     # the form for larger lattices
    say("transpose sites=%d pitch=%d %s" % (sites, pitch, dtype))
    x = torch.randn((sites, 36), dtype=dtype, device=dev())
    planes = torch.zeros((36, pitch), dtype=dtype, device=dev())
    stream = torch.cuda.current_stream().cuda_stream
    assert abi.su3_aos_to_soa_pitched(x.data_ptr(), planes.data_ptr(), sites, pitch, form, stream) == 0
    torch.cuda.synchronize()
    assert torch.equal(planes[:, :sites], x.t())
    assert int(torch.count_nonzero(planes[:, sites:])) == 0
    back = torch.empty_like(x)
    assert abi.su3_soa_to_aos_pitched(planes.data_ptr(), back.data_ptr(), sites, pitch, form, stream) == 0
    torch.cuda.synchronize()
    assert torch.equal(back, x)
