"""The standalone solve on arrays that are aligned to their elements only: views offset by one element
into their buffers, right-hand side, wall data and result, give the bits of the aligned solve."""
from __future__ import annotations

import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", [64, 32])
@pytest.mark.parametrize("bc", ["neumann", "dirichlet", "face_dirichlet"])
def test_solve_of_offset_views(bc, precision):
    import torch
    import paper_2111_04577_amd as drpf
    cfg = W.config("C2", nx=32, ny=8, nz=16, lx=1.0, ly=0.25, lz=0.5)
    print(f"[gpu] solve of offset views {bc} FP{precision}", flush=True)
    g = drpf.Grid(cfg, precision)
    dt = g.torch_dtype
    gen = torch.Generator(device="cuda").manual_seed(5)

    def offset(a):
        buf = torch.full((a.numel() + 3,), 7.0, dtype=dt, device="cuda")
        v = buf[1:1 + a.numel()].view(a.shape)
        v.copy_(a)
        return buf, v

    rhs = torch.randn(g.coarse_shape, dtype=dt, device="cuda", generator=gen)
    wall = torch.randn((2,) + g.coarse_shape[1:], dtype=dt, device="cuda", generator=gen)
    for w in (None, wall):
        ref = g.helmholtz_solve(rhs, "coarse", bc, 0.8, 90.0, wall=w)
        _, r = offset(rhs)
        ow = None if w is None else offset(w)[1]
        for solve in (g.helmholtz_solve, g.helmholtz_solve_static):
            buf, x = offset(torch.zeros_like(rhs))
            solve(r, "coarse", bc, 0.8, 90.0, out=x, wall=ow)
            torch.cuda.synchronize()
            assert x.data_ptr() % (2 * x.element_size()) != 0
            assert torch.equal(x, ref)
            assert float(buf[0]) == 7.0 and float(buf[-1]) == 7.0 and float(buf[-2]) == 7.0
