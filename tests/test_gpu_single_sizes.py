"""GPU parity of the single-resolution restricted set (G, densities, viscosities) formed in one march,
at the edges of its blocks: the smallest grid, tiles narrower than a wavefront, one and several
tiles across, relaxed walls. One step against the FP64 oracle: the velocity carries every face and
edge quantity. FP64 1e-10 of the largest entry (round-off of a stiff solve)."""
from __future__ import annotations

import numpy as np
import pytest

import workloads as W
from oracle import model
from oracle import step as S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,nz,over", [(4, 4, 4, {}), (16, 4, 8, {"d_w": 0.1}), (32, 16, 32, {}), (64, 8, 4, {}),
                                           (128, 16, 8, {"d_w": 0.1})])
def test_single_sizes(nx, ny, nz, over):
    import torch
    import paper_2111_04577_amd as drpf
    h = 1.0 / 16
    cfg = W.config("C2", nx=nx, ny=ny, nz=nz, lx=h * nx, ly=h * ny, lz=h * nz, radius=3.0 * h, noise=1e-3, seed=nx + nz,
                   refine=1, rho_ratio=10.0, mu_ratio=5.0, theta_bottom_deg=60.0, **over)
    print(f"[gpu] single resolution {nx} x {ny} x {nz} {over}", flush=True)
    ref = S.run(model.Params.from_config(cfg), W.droplet_state(cfg), 1)
    g = drpf.Grid(cfg, 64)
    d = g.state(W.droplet_state(cfg))
    g.step(d, 1)
    torch.cuda.synchronize()
    out = d.to_host()
    big = max(float(np.max(np.abs(ref[k][0]))) for k in "uvw")
    for k in "uvw":
        err = float(np.max(np.abs(out[k][0] - ref[k][0])))
        assert err <= 1e-10 * big, (k, err, big)
