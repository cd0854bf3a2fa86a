"""The conversions on both sides of the output sizes at which their stores change
policy, bit for bit against torch: a pack rounds to nearest even, an unpack is
exact, and with integer entries in [-9, 9] so is the rebuilt third row."""

import pytest
import torch

from _gpu import dev, guards_intact, poisoned, say

pytestmark = pytest.mark.gpu

WRITTEN = {("pack", "r12_f32"): 192, ("pack", "r12_f64"): 384, ("unpack", "r12_f32"): 576, ("unpack", "r12_f64"): 576,
           ("unpack", "bf16"): 576}
LINES = [144000000, 155000000, 286000000, 750000000]
CASES = [(op, f, line // n + past) for (op, f), n in WRITTEN.items() for line in LINES for past in (0, 1)]


@pytest.mark.parametrize("op,form,sites", CASES)
def test_either_side_of_a_line(op, form, sites):
    from paper_2103_00571_amd import abi

    say("%s %s sites=%d" % (op, form, sites))
    gen = torch.Generator(device="cuda")
    gen.manual_seed(sites)
    if op == "pack":
        src = torch.randn((sites, 4, 3, 3), dtype=torch.complex128, device=dev(), generator=gen)
        want = src[:, :, :2].to(torch.complex64 if form == "r12_f32" else torch.complex128)
    elif form == "bf16":
        src = torch.randn((sites, 4, 3, 3, 2), dtype=torch.float32, device=dev(), generator=gen).to(torch.bfloat16)
        want = torch.view_as_complex(src.to(torch.float64))
    else:
        z = torch.randint(-9, 10, (sites, 4, 2, 3, 2), device=dev(), generator=gen).to(torch.float64)
        rows = torch.view_as_complex(z)
        third = torch.linalg.cross(rows[:, :, 0], rows[:, :, 1]).conj().resolve_conj()
        want = torch.cat([rows, third[:, :, None]], dim=2)
        src = rows.to(torch.complex64) if form == "r12_f32" else rows
    out, whole = poisoned(want.shape, want.dtype)
    assert getattr(abi, "su3_" + op)(src.data_ptr(), out.data_ptr(), sites, getattr(abi, "SU3_" + form.upper()),
                                     torch.cuda.current_stream().cuda_stream) == 0
    torch.cuda.synchronize()
    assert torch.equal(out, want)
    assert guards_intact(whole)
