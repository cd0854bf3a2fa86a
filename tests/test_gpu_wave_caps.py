"""Calls on either side of the traffic where a kernel changes its occupancy
cap: a lattice taken in one call equals, bit for bit, the same lattice taken in
pieces that stay below every such limit."""

import pytest
import torch

from _gpu import dev, say

pytestmark = pytest.mark.gpu

# (and of the traffic where the stores change their cache policy)
# call, form, bytes per site read from a and written to c, limits in bytes
CASES = [
    ("nn", "SU3_F64", 576, 576, [192000000, 600000000]),
    ("nn", "SU3_BF16", 144, 144, [192000000, 600000000]),
    ("nn", "SU3_R12_F32", 192, 288, [160000000, 200000000, 600000000]),
    ("an", "SU3_F64", 576, 576, [600000000]),
    ("an", "SU3_F32", 288, 288, [600000000]),
    ("mat_vec", "SU3_F64", 576, 192, [400000000, 408000000, 1200000000]),
    ("mat_vec", "SU3_F32", 288, 96, [400000000, 1200000000]),
    ("pack", "SU3_R12_F32", 576, 192, [260000000, 1500000000]),
    ("pack", "SU3_R12_F64", 576, 384, [360000000, 600000000, 700000000]),
    ("unpack", "SU3_R12_F64", 384, 576, [130000000]),
]
CASES = [(op, form, na, nc, limit, past) for op, form, na, nc, limits in CASES
         for limit in limits for past in (0, 1)]


@pytest.mark.parametrize("op,form,na,nc,limit,past", CASES)
def test_either_side_of_a_cap(op, form, na, nc, limit, past):
    from paper_2103_00571_amd import abi

    nv = na // 12 if op == "mat_vec" else 0
    sites = limit // (na + nc + nv) + past
    say("%s %s sites=%d" % (op, form, sites))
    f = getattr(abi, form)
    real = torch.float64 if "F64" in form or op == "pack" else torch.float32
    gen = torch.Generator(device="cuda")
    gen.manual_seed(sites)
    if form == "SU3_BF16":
        real = torch.bfloat16
    a = torch.randn(sites * na // real.itemsize, dtype=real, device=dev(), generator=gen).view(torch.uint8)
    b = torch.randn(72, dtype=torch.float64 if "F64" in form else torch.float32, device=dev(), generator=gen)
    v = torch.randn(max(sites * nv // real.itemsize, 1), dtype=real, device=dev(), generator=gen).view(torch.uint8)
    stream = torch.cuda.current_stream().cuda_stream

    def run(out, s0, n):
        pa, pc, pv = a.data_ptr() + s0 * na, out.data_ptr() + s0 * nc, v.data_ptr() + s0 * nv
        if op == "nn":
            return abi.su3_mult_nn(pa, b.data_ptr(), pc, n, f, stream)
        if op == "an":
            return abi.su3_mult_an(pa, b.data_ptr(), pc, n, f, stream)
        if op == "mat_vec":
            return abi.su3_mat_vec(pa, pv, pc, n, f, stream)
        return (abi.su3_pack if op == "pack" else abi.su3_unpack)(pa, pc, n, f, stream)

    whole = torch.zeros(sites * nc, dtype=torch.uint8, device=dev())
    parts = torch.zeros_like(whole)
    assert run(whole, 0, sites) == 0
    step = 100000
    for s0 in range(0, sites, step):
        assert run(parts, s0, min(step, sites - s0)) == 0
    torch.cuda.synchronize()
    assert torch.equal(whole, parts)
    assert int(torch.count_nonzero(whole.view(torch.int64)[-nc // 8:])) > 0


# Where the plain copy changes its stores (6,144 KiB) and its cap (600 MB of
# traffic), with a ragged last workgroup.
@pytest.mark.parametrize("nbytes", [6144 * 1024 - 16, 6144 * 1024, 6144 * 1024 + 16, 300000000, 300000016])
def test_copy_on_either_side(nbytes):
    from paper_2103_00571_amd import ops

    say("copy of %d bytes" % nbytes)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(nbytes)
    src = torch.randint(0, 256, (nbytes,), dtype=torch.uint8, device=dev(), generator=gen)
    whole = torch.full((nbytes + 4096,), 7, dtype=torch.uint8, device=dev())
    ops.stream_copy(src, whole[2048:2048 + nbytes])
    torch.cuda.synchronize()
    assert torch.equal(whole[2048:2048 + nbytes], src)
    assert bool((whole[:2048] == 7).all()) and bool((whole[2048 + nbytes:] == 7).all())
