"""Calls on either side of the grids that are launched without an occupancy cap,
as a share of what the chip holds at once (24 wavefronts per CU, or what LDS
allows: 16 or 17 workgroups of 9 KiB). The entries are integers in [-9, 9], so every
form must equal torch's complex128 product (pack: its rows) bit for bit."""

import pytest
import torch

from _gpu import dev, guards_intact, ints, poisoned, say

pytestmark = pytest.mark.gpu

# call, form, sites at which the chip is full, share
CASES = [("nn", "f64", 32768, 75), ("na", "f64", 32768, 75), ("nn", "f32", 65536, 85), ("na", "f32", 65536, 85),
         ("nn", "r12c_f32", 98304, 85), ("an", "f64", 65536, 75), ("an", "f32", 131072, 92), ("an", "f32", 139264, 92),
         ("pack", "r12_f64", 65536, 75), ("pack", "r12_f64", 69632, 75)]
CASES = [(op, f, full * share // 100 + off) for op, f, full, share in CASES for off in (-16, 0, 1, 17)]


def _mm(x, y):
    return sum(x[..., :, m, None] * y[..., None, m, :] for m in range(3))


@pytest.mark.parametrize("op,form,sites", CASES)
def test_either_side_of_a_full_chip(op, form, sites):
    from paper_2103_00571_amd import abi

    say("%s %s sites=%d" % (op, form, sites))
    gen = torch.Generator(device="cuda")
    gen.manual_seed(sites)
    wide = torch.complex128 if form.endswith("f64") else torch.complex64
    a, b = ints((sites, 4, 2 if form == "r12c_f32" else 3, 3), gen), ints((4, 3, 3), gen)
    bh = b.transpose(-1, -2).conj().resolve_conj()
    if op == "pack":
        want = a[:, :, :2].contiguous()
    elif op == "an":
        want = _mm(a.transpose(-1, -2).conj().resolve_conj(), b).to(wide)
    else:
        want = _mm(a, bh if op == "na" else b).to(wide)
    x, y = a.to(wide), b.to(wide)
    out, whole = poisoned(want.shape, want.dtype)
    args = [x.data_ptr(), y.data_ptr(), out.data_ptr(), sites, getattr(abi, "SU3_" + form.upper()),
            torch.cuda.current_stream().cuda_stream]
    if op == "pack":
        del args[1]
    assert getattr(abi, "su3_pack" if op == "pack" else "su3_mult_" + op)(*args) == 0
    torch.cuda.synchronize()
    assert torch.equal(out, want)
    assert guards_intact(whole)
