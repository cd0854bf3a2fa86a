"""The SoA product where the planes do and do not start on 128-byte lines, at
the site counts where its windows begin and end. With integer entries in
[-9, 9] every operation is exact in FP32 and FP64, so the product must equal
torch's complex128 product bit for bit; the padding and everything around the
planes stay untouched."""

import pytest
import torch

from _gpu import dev, say

pytestmark = pytest.mark.gpu

SITES = [1, 7, 8, 15, 16, 17, 247, 248, 249, 256, 495, 496, 497, 512, 513, 993, 4097, 100003]


def _ints(shape, gen):
    z = torch.randint(-9, 10, (*shape, 2), device=dev(), generator=gen).to(torch.float64)
    return torch.view_as_complex(z)


@pytest.mark.parametrize("offset", [0, 16, 96])    # bytes of c's planes past a 128-byte line
@pytest.mark.parametrize("dtype", [torch.complex128, torch.complex64])
@pytest.mark.parametrize("sites", SITES)
def test_product_on_and_off_lines(sites, dtype, offset):
    from paper_2103_00571_amd import abi

    form, es = (abi.SU3_F64, 16) if dtype == torch.complex128 else (abi.SU3_F32, 8)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(sites)
    a, b = _ints((4, 3, 3, sites), gen), _ints((4, 3, 3), gen)
    want = sum(a[:, :, m, None, :] * b[:, None, m, :, None] for m in range(3)).to(dtype).reshape(36, sites)
    bt = b.to(dtype)
    stream = torch.cuda.current_stream().cuda_stream
    for pitch in sorted({sites, sites + 1, sites + 3, (sites + 15) // 16 * 16}):
        say("soa product sites=%d pitch=%d %s offset=%d" % (sites, pitch, dtype, offset))
        src = torch.full((36, pitch), float("nan"), dtype=dtype, device=dev())
        src[:, :sites] = a.reshape(36, sites)
        lead = offset // es
        whole = torch.full((lead + 36 * pitch + 64,), float("nan"), dtype=dtype, device=dev())
        out = whole[lead:lead + 36 * pitch].view(36, pitch)
        assert out.data_ptr() % 128 == offset
        assert abi.su3_mult_nn_soa_pitched(src.data_ptr(), bt.data_ptr(), out.data_ptr(), sites, pitch, form,
                                           stream) == 0
        torch.cuda.synchronize()
        assert torch.equal(out[:, :sites], want)
        assert int(torch.isnan(whole.real).sum()) == whole.numel() - 36 * sites
