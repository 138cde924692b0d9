"""GPU parity of the 2D restriction and chemical potential at the edges of its blocks: the fewest
columns and layers, one block, two and eight blocks across, relaxed walls. One step against the FP64 oracle: the velocity carries G, the densities and the viscosities
of every face and edge. 1e-10 of the largest entry (round-off of a stiff solve)."""
from __future__ import annotations

import numpy as np
import pytest

import workloads as W
from oracle import model
from oracle import step as S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,nz,over", [(4, 4, {}), (32, 4, {"d_w": 0.1}), (64, 8, {}), (16, 128, {"d_w": 0.1}),
                                        (256, 256, {})])
def test_restrict_2d_sizes(nx, nz, over):
    import torch
    import paper_2111_04577_amd as drpf
    h = 1.0 / 16
    cfg = W.config("C1", nx=nx, ny=1, nz=nz, lx=h * nx, ly=h, lz=h * nz, radius=3.0 * h, noise=1e-3, seed=nx + nz,
                   rho_ratio=10.0, mu_ratio=5.0, theta_bottom_deg=60.0, **over)
    print(f"[gpu] 2D restriction {nx} x {nz} {over}", flush=True)
    ref = S.run(model.Params.from_config(cfg), W.droplet_state(cfg), 1)
    g = drpf.Grid(cfg, 64)
    d = g.state(W.droplet_state(cfg))
    g.step(d, 1)
    torch.cuda.synchronize()
    out = d.to_host()
    big = max(float(np.max(np.abs(ref[k][0]))) for k in "uw")
    for k in "uw":
        err = float(np.max(np.abs(out[k][0] - ref[k][0])))
        assert err <= 1e-10 * big, (k, err, big)
