"""The adjoint where the end of dC or a is not finite. dA of a row depends on
that row of dC alone, and dB of a link on that link's rows alone, so an infinity
or NaN in the last link of the last site must leave the other three links of dB
as they are: the lanes past the end of a ragged lattice read those values again
and must add nothing. The entries are integers in [-9, 9], so every sum is exact
and the finite part must equal torch's complex128 contractions."""

import pytest
import torch

from _gpu import dev, ints, say

pytestmark = pytest.mark.gpu

# a ragged count for every launch form of both precisions, and whole tiles
SIZES = [1, 5, 15, 16, 17, 63, 8193, 16385, 32769, 100003, 131073, 400001, 700001]


@pytest.mark.parametrize("dtype", [torch.complex128, torch.complex64])
@pytest.mark.parametrize("sites", SIZES)
def test_last_link_does_not_reach_the_others(sites, dtype):
    from paper_2103_00571_amd import abi, ops

    form = abi.SU3_F64 if dtype == torch.complex128 else abi.SU3_F32
    gen = torch.Generator(device="cuda")
    gen.manual_seed(sites)
    a, dc, b = (ints(s, gen) for s in ((sites, 4, 3, 3), (sites, 4, 3, 3), (4, 3, 3)))
    da = sum(dc[..., :, m, None] * b.conj()[None, :, None, :, m] for m in range(3)).to(dtype)
    db = sum((a.conj()[:, :, m, :, None] * dc[:, :, m, None, :]).sum(0) for m in range(3))
    inf, nan = float("inf"), float("nan")
    # the last chunk of an array is its last complex value in FP64, its last two in FP32
    for where, at, value in (("dc", 2, complex(nan, nan)), ("dc", 2, complex(0.0, -inf)), ("dc", 1, complex(inf, 1.0)),
                             ("a", 2, complex(nan, inf))):
        say("adjoint sites=%d %s %s in the last row of %s" % (sites, dtype, value, where))
        x, g = a.to(dtype, copy=True), dc.to(dtype, copy=True)
        (g if where == "dc" else x)[-1, 3, 2, at] = value
        oa, ob = ops.mult_nn_bwd(x, b.to(dtype), g)
        ws = ops.mult_nn_bwd_workspace(sites, form, dev())
        alone = torch.full((4, 3, 3), nan, dtype=dtype, device=dev())
        stream = torch.cuda.current_stream().cuda_stream
        assert abi.su3_mult_nn_grad(x.data_ptr(), None, g.data_ptr(), None, alone.data_ptr(), sites, form,
                                    ws.data_ptr(), ws.numel(), stream) == 0
        torch.cuda.synchronize()
        for got, want in ((ob, db), (alone, db.to(dtype))):
            assert torch.equal(got[:3], want[:3])
            # column `at` of dC (row `at` of dB from a) takes the value in, the rest does not
            hit = got[3, :, at] if where == "dc" else got[3, at, :]
            assert not bool(torch.isfinite(torch.view_as_real(hit)).all(-1).any())
            keep = [i for i in range(3) if i != at]
            assert torch.equal(got[3][:, keep] if where == "dc" else got[3][keep],
                               want[3][:, keep] if where == "dc" else want[3][keep])
        assert torch.equal(oa.flatten(0, 2)[:-1], da.flatten(0, 2)[:-1])
        if where == "dc":
            assert not bool(torch.isfinite(torch.view_as_real(oa[-1, 3, 2])).all(-1).any())
        else:
            assert torch.equal(oa, da)
