"""The adjoint's workspace sizes, which need no GPU: the size that a call must
have stays what callers may have kept (72 FP64 partials for every 12 tiles of 64
rows, and one more set for every 2,048 of those), the size for the best speed is
at least that, and both grow with the lattice."""

import pytest


@pytest.fixture(scope="module")
def abi():
    from paper_2103_00571_amd import abi
    return abi


A, B, D, DA, DB, WS = (1 << k for k in (38, 40, 41, 42, 43, 44))
SIZES = sorted({1, 5, 63, 64, 65, 1000, 4096, 8193, 16384, 16385, 32768, 32769, 65536, 65537, 131072, 131073,
                400000, 400001, 700000, 800001, 48 ** 4, 7 * 10 ** 6} | {10 ** k for k in range(8)})


def _smallest(sites):
    tiles = -(-12 * sites // 64)
    groups = -(-tiles // 12)
    return 576 * (groups + -(-groups // 2048))


@pytest.mark.parametrize("form", [0, 1])
def test_workspace_sizes(abi, form):
    need = [abi.su3_mult_nn_bwd_workspace_bytes(n, form) for n in SIZES]
    best = [abi.su3_mult_nn_bwd_workspace_best_bytes(n, form) for n in SIZES]
    assert need == [_smallest(n) for n in SIZES]
    assert all(n <= b <= 4 * n + 576 for n, b in zip(need, best))
    assert best == sorted(best) and need == sorted(need)
    assert abi.su3_mult_nn_bwd_workspace_best_bytes(0, form) == 0
    assert abi.su3_mult_nn_bwd_workspace_best_bytes(1000, 2) == 0


@pytest.mark.parametrize("form", [0, 1])
def test_less_than_the_smallest_is_refused(abi, form):
    for n in SIZES:
        need = _smallest(n)
        assert abi.su3_mult_nn_bwd(A, B, D, DA, DB, n, form, WS, need - 8, None) == abi.SU3_ERR_WORKSPACE
        assert abi.su3_mult_nn_grad(A, None, D, None, DB, n, form, WS, need - 8, None) == abi.SU3_ERR_WORKSPACE
        # inside the part that every form writes
        assert abi.su3_mult_nn_bwd(A, B, D, WS + need - 16, DB, n, form, WS, 1 << 30, None) == abi.SU3_ERR_OVERLAP
