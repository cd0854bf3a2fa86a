"""FP32 and BF16 pack and unpack at the ends of their tiles and on both sides
of the size at which a grid stops fitting on the chip at once, bit for bit
against torch's conversions, with nothing written around the output."""

import pytest
import torch

from _gpu import dev, guards_intact, poisoned, say

pytestmark = pytest.mark.gpu

SITES = [1, 7, 8, 14, 15, 57, 64, 65, 43690, 43691, 100003]


@pytest.mark.parametrize("form", ["f32", "bf16"])
@pytest.mark.parametrize("sites", SITES)
def test_pack_and_unpack(sites, form):
    from paper_2103_00571_amd import abi

    say("pack/unpack sites=%d %s" % (sites, form))
    gen = torch.Generator(device="cuda")
    gen.manual_seed(sites)
    wide = torch.randn((sites, 4, 3, 3, 2), dtype=torch.float64, device=dev(), generator=gen)
    code, dtype = (abi.SU3_F32, torch.float32) if form == "f32" else (abi.SU3_BF16, torch.bfloat16)
    want = wide.to(torch.float32).to(dtype)
    stream = torch.cuda.current_stream().cuda_stream
    out, whole = poisoned((sites, 4, 3, 3, 2), dtype)
    assert abi.su3_pack(wide.data_ptr(), out.data_ptr(), sites, code, stream) == 0
    torch.cuda.synchronize()
    assert torch.equal(out.view(torch.int16), want.view(torch.int16)) and guards_intact(whole)
    back, whole = poisoned((sites, 4, 3, 3, 2), torch.float64)
    assert abi.su3_unpack(want.data_ptr(), back.data_ptr(), sites, code, stream) == 0
    torch.cuda.synchronize()
    assert torch.equal(back, want.to(torch.float64)) and guards_intact(whole)
