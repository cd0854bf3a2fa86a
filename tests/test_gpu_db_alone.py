"""dB where stage 2 adds several runs, alone (su3_mult_nn_grad without dA, past
1,048,576 FP64 and 2,097,152 FP32 sites) and with dA, on data that is not integer
and cancels: half of the sites repeat the other half with -dC, so dB is the sum
over a few last sites while the sum of magnitudes stays that of the whole lattice.
A sum in FP32, or one that takes a partial twice, is off by far more than the bound:
every component is a sum of fewer than 512 roundings deep in FP64 (64 or 128 fused
multiply-adds per lane, then 9 + 9 + 18 + 70 additions), so its error is at most
512 * 2^-53 times the sum of magnitudes; FP32 dB is rounded once more, by at most
2^-24 of its value. Repeated calls on a dirty workspace agree bit for bit."""

import pytest
import torch

from _gpu import dev, say

pytestmark = pytest.mark.gpu

CASES = [(torch.complex128, n) for n in (1048576, 1048577, 1600001)]
CASES += [(torch.complex64, n) for n in (2097152, 2097153, 2500007)]


@pytest.mark.parametrize("dtype,sites", CASES)
def test_db_of_many_runs(dtype, sites):
    from paper_2103_00571_amd import abi, ops

    say("db of many runs sites=%d %s" % (sites, dtype))
    form = abi.SU3_F64 if dtype == torch.complex128 else abi.SU3_F32
    gen = torch.Generator(device="cuda")
    gen.manual_seed(sites)
    half, rest = (sites - 5) // 2, sites - 2 * ((sites - 5) // 2)
    x, g = (torch.randn((half + rest, 4, 3, 3), dtype=dtype, device=dev(), generator=gen) for _ in range(2))
    a, dc = torch.cat([x[:half], x]), torch.cat([-g[:half], g])
    b = torch.randn((4, 3, 3), dtype=dtype, device=dev(), generator=gen)
    xe, ge = x[half:].to(torch.complex128), g[half:].to(torch.complex128)
    want = sum((xe.conj()[:, :, m, :, None] * ge[:, :, m, None, :]).sum(0) for m in range(3))
    big = torch.zeros((4, 3, 3), dtype=torch.float64, device=dev())
    for s0 in range(0, sites, 1 << 18):
        p = torch.view_as_real(a[s0:s0 + (1 << 18)].to(torch.complex128)).abs().sum(-1)
        q = torch.view_as_real(dc[s0:s0 + (1 << 18)].to(torch.complex128)).abs().sum(-1)
        big += sum((p[:, :, m, :, None] * q[:, :, m, None, :]).sum(0) for m in range(3))
    bound = 512 * 2.0 ** -53 * big
    ws = ops.mult_nn_bwd_workspace(sites, form, dev())
    ws.fill_(0xff)
    stream = torch.cuda.current_stream().cuda_stream
    seen = []
    for _ in range(3):
        alone = torch.full((4, 3, 3), float("nan"), dtype=dtype, device=dev())
        assert abi.su3_mult_nn_grad(a.data_ptr(), None, dc.data_ptr(), None, alone.data_ptr(), sites, form,
                                    ws.data_ptr(), ws.numel(), stream) == 0
        both = torch.full((4, 3, 3), float("nan"), dtype=dtype, device=dev())
        da = torch.empty_like(a)
        assert abi.su3_mult_nn_grad(a.data_ptr(), b.data_ptr(), dc.data_ptr(), da.data_ptr(), both.data_ptr(), sites,
                                    form, ws.data_ptr(), ws.numel(), stream) == 0
        _, wide = ops.mult_nn_bwd(a, b, dc, da=da, ws=ws)
        torch.cuda.synchronize()
        seen.append((alone, both, wide))
        for got in (alone, both, wide):
            err = torch.view_as_real(got.to(torch.complex128) - want).abs()
            once = 0.0 if got.dtype == torch.complex128 else 2.0 ** -24
            assert bool((err <= bound[..., None] + once * torch.view_as_real(want).abs()).all())
        # with dA the two entries sum in one order: FP32 dB is the FP64 one rounded once
        assert torch.equal(both, wide.to(dtype))
    for later in seen[1:]:
        assert all(torch.equal(p, q) for p, q in zip(seen[0], later))
