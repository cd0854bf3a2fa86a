"""Argument validation of su3_mult_nn_grad, which needs no GPU: as
su3_mult_nn_bwd with da, and without it da and b are not looked at."""

import pytest


@pytest.fixture(scope="module")
def abi():
    from paper_2103_00571_amd import abi
    return abi


A, B, D, DA, DB, WS = (1 << k for k in (38, 40, 41, 42, 43, 44))


def test_grad_validation(abi):
    f = abi.su3_mult_nn_grad
    for form in (abi.SU3_F64, abi.SU3_F32):
        need = abi.su3_mult_nn_bwd_workspace_bytes(1000, form)
        size = 1000 * (576 if form == abi.SU3_F64 else 288)
        assert f(A, B, D, DA, DB, 1000, abi.SU3_BF16, WS, need, None) == abi.SU3_ERR_PRECISION
        for da, b in ((DA, B), (None, None)):
            assert f(A, b, D, da, DB, -1, form, WS, need, None) == abi.SU3_ERR_SIZE
            assert f(A, b, D, da, None, 1000, form, WS, need, None) == abi.SU3_ERR_NULL
            assert f(None, b, D, da, DB, 1000, form, WS, need, None) == abi.SU3_ERR_NULL
            assert f(A, b, None, da, DB, 1000, form, WS, need, None) == abi.SU3_ERR_NULL
            assert f(A, b, D, da, None, 0, form, None, 0, None) == abi.SU3_ERR_NULL
            assert f(A, b, D, da, DB, 1000, form, WS, need - 8, None) == abi.SU3_ERR_WORKSPACE
            assert f(A, b, D, da, DB, 1000, form, None, need, None) == abi.SU3_ERR_WORKSPACE
            assert f(A + 8, b, D, da, DB, 1000, form, WS, need, None) == abi.SU3_ERR_ALIGN
            assert f(A, b, D + 8, da, DB, 1000, form, WS, need, None) == abi.SU3_ERR_ALIGN
            assert f(A, b, D, da, DB, 1000, form, WS + 8, need, None) == abi.SU3_ERR_ALIGN
            assert f(A, b, D, da, DB + 2, 1000, form, WS, need, None) == abi.SU3_ERR_ALIGN
            assert f(A, b, D, da, A + size - 8, 1000, form, WS, need, None) == abi.SU3_ERR_OVERLAP
            assert f(A, b, D, da, D, 1000, form, WS, need, None) == abi.SU3_ERR_OVERLAP
            assert f(A, b, D, da, DB, 1000, form, A, need, None) == abi.SU3_ERR_OVERLAP
            assert f(A, b, D, da, DB, 1000, form, D, need, None) == abi.SU3_ERR_OVERLAP
            assert f(A, b, D, da, WS + 16, 1000, form, WS, need, None) == abi.SU3_ERR_OVERLAP
        assert f(A, None, D, DA, DB, 1000, form, WS, need, None) == abi.SU3_ERR_NULL
        assert f(A, B, D, A, DB, 1000, form, WS, need, None) == abi.SU3_ERR_OVERLAP
        assert f(A, B, D, DA, DA + 64, 1000, form, WS, need, None) == abi.SU3_ERR_OVERLAP
        assert f(A, B, D, DA + 8, DB, 1000, form, WS, need, None) == abi.SU3_ERR_ALIGN
        assert f(A, WS + 64, D, DA, DB, 1000, form, WS, need, None) == abi.SU3_ERR_OVERLAP
