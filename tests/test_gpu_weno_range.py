"""Range of the FP32 WENO-Z face values: a patch of uniform polymer stress beside a jump, where three
upwind cells are equal and the weight of that candidate reaches 8 jump^2 / eps, its product with the value V
about V jump^2 / eps: in range for V jump^2 < 4e8. One step of the 3D stress
form on an FP32 grid against the FP64 oracle, with the jump along each axis. Storage and update
round-off: 32 eps_32 = 4e-6 of the largest stress (the step changes it by less than its size)."""
from __future__ import annotations

import numpy as np
import pytest

import workloads as W
from oracle import model
from oracle import step as S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("axis", [0, 1, 2])
@pytest.mark.parametrize("low,high", [(0.5, 1.0), (200.0, 400.0), (1.0, 601.0)])
def test_fp32_weno_beside_a_jump(low, high, axis):
    import torch
    import paper_2111_04577_amd as drpf
    n = 16
    h = 1.0 / n
    cfg = W.config("C3", nx=n, ny=n, nz=n, lx=1.0, ly=1.0, lz=1.0, radius=0.3, cn=2.0 * h, dt=1e-5, advection=1)
    print(f"[gpu] FP32 WENO-Z beside a jump {low} -> {high} along axis {axis}", flush=True)
    st = W.droplet_state(cfg)
    # a smooth flow through every face of the jump, both signs
    k = 2.0 * np.pi * (np.arange(n) + 0.5) * h
    z, y, x = np.meshgrid(k, k, k, indexing="ij")
    st["u"] = [np.sin(y) + 0.5 * np.cos(z)] * 2
    st["v"] = [np.sin(x) + 0.5 * np.cos(z)] * 2
    w = np.sin(x) * np.cos(y)
    w[-1] = 0.0
    st["w"] = [w] * 2
    half = np.where(np.arange(n) < n // 2, low, high).reshape([-1 if a == axis else 1 for a in range(3)])
    tau = np.broadcast_to(half, (n, n, n)).astype(np.float32).astype(np.float64)
    st["tau"] = [[np.array(tau) for _ in range(6)] for _ in range(2)]
    ref = S.run(model.Params.from_config(cfg), st, 1)
    g = drpf.Grid(cfg, 32)
    d = g.state(st)
    g.step(d, 1)
    torch.cuda.synchronize()
    out = d.to_host()["tau"][0]
    for m in range(6):
        assert np.all(np.isfinite(out[m])), m
        err = float(np.max(np.abs(out[m] - ref["tau"][0][m])))
        assert err <= 32 * 2.0 ** -23 * high, (m, err)
