"""The adjoint and dB alone in each of the two workspace sizes, on both sides of
every size at which the launch changes with them. Integer entries in [-9, 9] make
every sum exact, so dB must equal torch's complex128 sum whatever its order; the
workspace starts as NaN, is reused dirty, and nothing past the bytes given is
written."""

import pytest
import torch

from _gpu import dev, ints, say

pytestmark = pytest.mark.gpu

SIZES = [1, 63, 4096, 8193, 16384, 16385, 24577, 32768, 32769, 131072, 131073, 400000, 400001, 700001]


@pytest.mark.parametrize("dtype", [torch.complex128, torch.complex64])
@pytest.mark.parametrize("sites", SIZES)
def test_both_workspace_sizes(sites, dtype):
    from paper_2103_00571_amd import abi

    say("adjoint workspaces sites=%d %s" % (sites, dtype))
    form = abi.SU3_F64 if dtype == torch.complex128 else abi.SU3_F32
    gen = torch.Generator(device="cuda")
    gen.manual_seed(sites)
    a, dc, b = (ints(s, gen) for s in ((sites, 4, 3, 3), (sites, 4, 3, 3), (4, 3, 3)))
    da = sum(dc[..., :, m, None] * b.conj()[None, :, None, :, m] for m in range(3)).to(dtype)
    db = sum((a.conj()[:, :, m, :, None] * dc[:, :, m, None, :]).sum(0) for m in range(3))
    a, dc, b = a.to(dtype), dc.to(dtype), b.to(dtype)
    stream = torch.cuda.current_stream().cuda_stream
    sizes = [abi.su3_mult_nn_bwd_workspace_bytes(sites, form), abi.su3_mult_nn_bwd_workspace_best_bytes(sites, form)]
    for need in sizes:
        ws = torch.full((need // 8 + 64,), float("nan"), dtype=torch.float64, device=dev())
        for _ in range(2):
            oa = torch.full_like(a, float("nan"))
            ob = torch.full((4, 3, 3), float("nan"), dtype=torch.complex128, device=dev())
            alone = torch.full((4, 3, 3), float("nan"), dtype=dtype, device=dev())
            assert abi.su3_mult_nn_bwd(a.data_ptr(), b.data_ptr(), dc.data_ptr(), oa.data_ptr(), ob.data_ptr(), sites,
                                       form, ws.data_ptr(), need, stream) == 0
            assert abi.su3_mult_nn_grad(a.data_ptr(), None, dc.data_ptr(), None, alone.data_ptr(), sites, form,
                                        ws.data_ptr(), need, stream) == 0
            torch.cuda.synchronize()
            assert torch.equal(oa, da) and torch.equal(ob, db) and torch.equal(alone, db.to(dtype))
        assert bool(torch.isnan(ws[need // 8:]).all())

    # an arena given as the workspace, with dA in it behind the smallest size
    arena = torch.full((sizes[0] // 8 + 2 * a.numel() * a.element_size() // 8 + 64,), float("nan"),
                       dtype=torch.float64, device=dev())
    oa = arena[sizes[0] // 8:].view(dtype)[:a.numel()].view(a.shape)
    ob.fill_(float("nan"))
    assert abi.su3_mult_nn_bwd(a.data_ptr(), b.data_ptr(), dc.data_ptr(), oa.data_ptr(), ob.data_ptr(), sites, form,
                               arena.data_ptr(), arena.numel() * 8, stream) == 0
    torch.cuda.synchronize()
    assert torch.equal(oa, da) and torch.equal(ob, db)
