"""The tile solvers of the general path at large orders, where they are bound by
the loads of the tile products: workgroups per CU, and a real solve of an order
that takes the variant for many tiles (above 4096)."""

import pytest

pytestmark = pytest.mark.gpu


# complex: 25 and 50 KB of LDS of 160; real: 96 registers of 512, and 154
@pytest.mark.parametrize("prec,cplx,least", [("fp32", 1, 6), ("fp64", 1, 3), ("fp32", 0, 5), ("fp64", 0, 3)])
def test_workgroups_per_cu(prec, cplx, least):
    from paper_2607_12430_amd import _lib
    assert _lib.lib().msqrt_test_tile_occupancy(_lib.PREC_NAMES[prec], cplx) >= least


@pytest.mark.parametrize("n", [4129, 4350])
def test_real_order_above_4096(n):
    import torch
    import paper_2607_12430_amd as msq
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    a = 2.0 * torch.eye(n, device="cuda", dtype=torch.float64)
    a += torch.randn(n, n, generator=g, device="cuda", dtype=torch.float64) / n ** 0.5
    print(f"[tile occupancy] real {n}", flush=True)
    x, info = msq.sqrtm(a, prec="fp32", fallback=False)
    # the corrections converge only if their Sylvester equations are solved
    assert info["status"] == "ok" and info["steps"] <= 3 and info["relres"] <= 1e-13
    r = torch.linalg.matrix_norm(x @ x - a) / torch.linalg.matrix_norm(a)
    assert float(r) <= 2e-13
