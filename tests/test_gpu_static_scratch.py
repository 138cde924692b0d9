"""The allocation-free solve needs its spectral buffer only, with wall data too: a solve whose spectral
buffer fits the 32 MiB scratch, but would not beside a right-hand side of its own, runs and gives
the bits of drpf_helmholtz_solve."""
from __future__ import annotations

import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bc", ["neumann", "dirichlet", "face_dirichlet"])
def test_static_solve_with_wall_data_near_the_limit(bc):
    import torch
    import paper_2111_04577_amd as drpf
    # 129 * 256 * 32 complex FP64 = 16.9 MB, the right-hand side 16.8 MB
    cfg = W.config("C2", nx=256, ny=256, nz=32, refine=1)
    print(f"[gpu] static solve near the limit {bc}", flush=True)
    g = drpf.Grid(cfg, 64)
    gen = torch.Generator(device="cuda").manual_seed(3)
    rhs = torch.randn(g.coarse_shape, dtype=torch.float64, device="cuda", generator=gen)
    wall = torch.randn((2,) + g.coarse_shape[1:], dtype=torch.float64, device="cuda", generator=gen)
    a = g.helmholtz_solve_static(rhs, "coarse", bc, 0.8, 900.0, wall=wall)
    b = g.helmholtz_solve(rhs, "coarse", bc, 0.8, 900.0, wall=wall)
    torch.cuda.synchronize()
    assert torch.equal(a, b)
