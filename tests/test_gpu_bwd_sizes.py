"""The adjoint on both sides of every size at which its launch changes: dA
and dB bit for bit. With integer entries in [-9, 9] every product and partial
sum is exact in FP32 (dA) and FP64 (dB), so both must equal torch's complex128
contractions. The workspace starts as NaN, is reused dirty, and nothing past
the bytes asked for is written."""

import pytest
import torch

from _gpu import dev, say

pytestmark = pytest.mark.gpu

SIZES = [1, 16384, 16385, 32768, 32769, 43690, 87382, 131072, 131073, 400000, 400001, 700000, 700001]


def _ints(shape, gen):
    z = torch.randint(-9, 10, (*shape, 2), device=dev(), generator=gen).to(torch.float64)
    return torch.view_as_complex(z)


@pytest.mark.parametrize("dtype", [torch.complex128, torch.complex64])
@pytest.mark.parametrize("sites", SIZES)
def test_adjoint_where_its_launch_changes(sites, dtype):
    from paper_2103_00571_amd import abi

    say("adjoint sites=%d %s" % (sites, dtype))
    form = abi.SU3_F64 if dtype == torch.complex128 else abi.SU3_F32
    gen = torch.Generator(device="cuda")
    gen.manual_seed(sites)
    a, dc, b = (_ints(s, gen) for s in ((sites, 4, 3, 3), (sites, 4, 3, 3), (4, 3, 3)))
    da = sum(dc[..., :, m, None] * b.conj()[None, :, None, :, m] for m in range(3)).to(dtype)
    db = sum((a.conj()[:, :, m, :, None] * dc[:, :, m, None, :]).sum(0) for m in range(3))
    at, dct, bt = a.to(dtype), dc.to(dtype), b.to(dtype)
    need = abi.su3_mult_nn_bwd_workspace_bytes(sites, form)
    ws = torch.full((need // 8 + 64,), float("nan"), dtype=torch.float64, device=dev())
    stream = torch.cuda.current_stream().cuda_stream
    for _ in range(3):
        oa = torch.full_like(at, float("nan"))
        ob = torch.full((4, 3, 3), float("nan"), dtype=torch.complex128, device=dev())
        assert abi.su3_mult_nn_bwd(at.data_ptr(), bt.data_ptr(), dct.data_ptr(), oa.data_ptr(), ob.data_ptr(), sites,
                                   form, ws.data_ptr(), need, stream) == 0
        torch.cuda.synchronize()
        assert torch.equal(oa, da)
        assert torch.equal(ob, db)
    assert bool(torch.isnan(ws[need // 8:]).all())


def test_a_workspace_serves_every_smaller_lattice():
    from paper_2103_00571_amd import abi

    for form in (abi.SU3_F64, abi.SU3_F32):
        sizes = sorted(set(SIZES) | {10 ** k for k in range(8)} | {s - 1 for s in SIZES if s > 1})
        need = [abi.su3_mult_nn_bwd_workspace_bytes(n, form) for n in sizes]
        assert need == sorted(need)
