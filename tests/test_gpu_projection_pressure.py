"""GPU parity of the pressure of the wall-normal projection by recurrences (3D FP64, deep or many
columns): its zero-mean (0,0) mode, four and eight rows per thread, one mode per block, a last block that
is not full, the deepest columns. One phase at rest, a rough velocity: one step against the FP64 oracle,
1e-10 of the largest pressure and of its mean's scale (round-off of a stiff solve)."""
from __future__ import annotations

import numpy as np
import pytest

import workloads as W
from oracle import model
from oracle import step as S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,nz", [(128, 64, 32), (64, 64, 64), (4, 4, 128), (8, 4, 256), (4, 4, 512)])
def test_projection_pressure(nx, ny, nz):
    import torch
    import paper_2111_04577_amd as drpf
    h = 1.0 / 16
    cfg = W.config("C2", nx=nx, ny=ny, nz=nz, lx=h * nx, ly=h * ny, lz=h * nz, radius=3.0 * h, seed=nz, rho_ratio=10.0,
                   mu_ratio=5.0)
    print(f"[gpu] projected pressure {nx} x {ny} x {nz}", flush=True)
    st = W.droplet_state(cfg)
    st["phi"] = [np.ones_like(a) for a in st["phi"]]
    for i, k in enumerate("uvw"):
        a = 2.0 * W.splitmix64_uniform(7 + i, nx * ny * nz).reshape(nz, ny, nx) - 1.0
        # w of the (0,0) mode: its divergence is the data of the singular pressure equation
        if k == "w":
            a += np.sin(np.arange(1, nz + 1) * (np.pi / nz)).reshape(-1, 1, 1)
            a[-1] = 0.0
        st[k] = [a, a.copy()]
    ref = S.run(model.Params.from_config(cfg), st, 1)["p"][0]
    g = drpf.Grid(cfg, 64)
    d = g.state(st)
    g.step(d, 1)
    torch.cuda.synchronize()
    out = d.to_host()["p"][0]
    big = float(np.max(np.abs(ref)))
    err, mean = float(np.max(np.abs(out - ref))), abs(float(np.mean(out)))
    print(f"[gpu] p: {err / big:.2e}, mean {mean / big:.2e}", flush=True)
    assert err <= 1e-10 * big, (err, big)
    assert mean <= 1e-10 * big, (mean, big)
