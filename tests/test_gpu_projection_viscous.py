"""GPU parity of the wall-normal velocity solves where the step is far longer than the diffusion time
of a cell: the gap of the (0,0) mode, gamma0 hz^2 / (dt nu), down to 1e-12. One phase whose
viscosity is half the implicit one, so that u^{n+1} is of the order of u^n; a shear profile, one step
against the FP64 oracle. The explicit viscous term holds round-off of order eps nu u / hz^2, which the
solve returns as eps nz^2 u: 8 eps nz^2 = 2e-12 at 32 rows. The forms of the pass change at 1e-3."""
from __future__ import annotations

import numpy as np
import pytest

import workloads as W
from oracle import model
from oracle import step as S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("gap", [1e-2, 2e-3, 5e-4, 1e-6, 1e-10, 1e-12])
@pytest.mark.parametrize("nx,ny,nz", [(128, 64, 32), (8, 4, 128)])
def test_projection_viscous(nx, ny, nz, gap):
    import torch
    import paper_2111_04577_amd as drpf
    h = 1.0 / 16
    dt = 1e-4
    re = 2.0 * dt * gap / h ** 2  # nu = 2 / Re, gamma0 = 1
    cfg = W.config("C2", nx=nx, ny=ny, nz=nz, lx=h * nx, ly=h * ny, lz=h * nz, rho_ratio=1.0, mu_ratio=0.5, re=re, dt=dt)
    print(f"[gpu] viscous projection {nx} x {ny} x {nz} gap {gap}", flush=True)

    def state():
        st = W.droplet_state(cfg)
        st["phi"] = [np.ones_like(a) for a in st["phi"]]
        z = ((np.arange(nz) + 0.5) / nz).reshape(-1, 1, 1)
        for k, a in (("u", 4.0 * z * (1.0 - z) + 0.3 * np.sin(3.0 * z)), ("v", np.cos(5.0 * z) - z)):
            f = np.broadcast_to(a, (nz, ny, nx))
            st[k] = [np.array(f), np.array(f)]
        return st

    ref = S.run(model.Params.from_config(cfg), state(), 1)
    g = drpf.Grid(cfg, 64)
    d = g.state(state())
    g.step(d, 1)
    torch.cuda.synchronize()
    out = d.to_host()
    for k in "uv":
        big = float(np.max(np.abs(ref[k][0])))
        err = float(np.max(np.abs(out[k][0] - ref[k][0])))
        print(f"[gpu] {k}: {err / big:.2e} of {big:.2e}", flush=True)
        assert err <= 8 * 2.0 ** -52 * nz ** 2 * big, (k, err, big)
