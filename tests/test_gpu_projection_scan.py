"""GPU parity of the wall-normal projection by recurrences (3D FP64, deep or many columns) at the edges of
its range: the shallowest columns it takes, one to 16 modes per block, a last block that is not
full, the deepest columns, moving walls, a single resolution. One phase at rest, a rough velocity:
one step against the FP64 oracle, FP64 1e-10 of the largest velocity (round-off of a stiff solve);
FP32 (cyclic reduction) 2e-5 (storage and transform round-off of a velocity of order one, 1e-6, and of the pressure
gradient that the rough velocity's divergence needs, some ten times that)."""
from __future__ import annotations

import numpy as np
import pytest

import workloads as W
from oracle import model
from oracle import step as S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,nz,over", [(4, 4, 128, {}), (8, 4, 256, {}), (4, 4, 512, {}), (64, 64, 64, {}),
                                           (128, 64, 32, {}), (16, 4, 128, {"refine": 1}),
                                           (8, 8, 128, {"u_wall_bottom": (0.3, -0.1), "u_wall_top": (-0.2, 0.4)})])
def test_projection_scan(nx, ny, nz, over):
    import torch
    import paper_2111_04577_amd as drpf
    h = 1.0 / 16
    cfg = W.config("C2", nx=nx, ny=ny, nz=nz, lx=h * nx, ly=h * ny, lz=h * nz, radius=3.0 * h, seed=nz, rho_ratio=10.0,
                   mu_ratio=5.0, **over)
    print(f"[gpu] projection {nx} x {ny} x {nz} {over}", flush=True)

    def state():
        st = W.droplet_state(cfg)
        st["phi"] = [np.ones_like(a) for a in st["phi"]]
        for i, k in enumerate("uvw"):
            a = 2.0 * W.splitmix64_uniform(7 + i, nx * ny * nz).reshape(nz, ny, nx) - 1.0
            if k == "w":
                a[-1] = 0.0
            st[k] = [a, a.copy()]
        return st

    ref = S.run(model.Params.from_config(cfg), state(), 1)
    big = max(float(np.max(np.abs(ref[k][0]))) for k in "uvw")
    for precision, tol in ((64, 1e-10), (32, 2e-5)):
        g = drpf.Grid(cfg, precision)
        d = g.state(state())
        g.step(d, 1)
        torch.cuda.synchronize()
        out = d.to_host()
        err = max(float(np.max(np.abs(out[k][0] - ref[k][0]))) for k in "uvw")
        assert err <= tol * big, (precision, err, big)
