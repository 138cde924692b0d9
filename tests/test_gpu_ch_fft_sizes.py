"""GPU parity of the fused Cahn-Hilliard right-hand side and x transform at the edges of its
blocks: the narrowest and widest rows it takes and their neighbours on either side, fewer rows than
a block holds, odd counts of layer batches, 2D, single resolution, given advection (WENO-Z) and
relaxed walls. Two steps (start-up and BDF2) against the FP64 oracle: FP64 1e-10 of the largest
entry (round-off of a stiff solve, as in every parity test here), FP32 phi 1e-4 (its 1e-6 of the
fourth-order right-hand side over two steps)."""
from __future__ import annotations

import numpy as np
import pytest

import workloads as W
from oracle import model
from oracle import step as S

pytestmark = pytest.mark.gpu

# base, (nx, ny, nz) of the flow grid, overrides
CASES = [
    ("C2", (4, 4, 4), {}),       # fine rows of 8: two passes
    ("C2", (8, 4, 4), {}),       # fine rows of 16: the narrowest
    ("C1", (8, 1, 4), {}),
    ("C2", (8, 32, 8), {}),      # eight rows per block
    ("C2", (16, 4, 16), {"advection": 1}),
    ("C2", (32, 8, 8), {"d_w": 0.1, "theta_bottom_deg": 60.0}),
    ("C1", (64, 1, 16), {"d_w": 0.1, "theta_bottom_deg": 60.0}),
    ("C2", (16, 8, 8), {"refine": 1, "d_w": 0.1}),
    ("C2", (256, 4, 4), {}),     # two FP64 rows per block
    ("C2", (512, 4, 4), {"d_w": 0.1}),  # FP32: two rows per block; FP64: two passes
    ("C1", (512, 1, 4), {}),     # one FP64 row of 512 threads
]


@pytest.mark.parametrize("base,n,over", CASES)
def test_ch_fft_sizes(base, n, over):
    import torch
    import paper_2111_04577_amd as drpf
    nx, ny, nz = n
    h = 1.0 / 16
    cfg = W.config(base, nx=nx, ny=ny, nz=nz, lx=h * nx, ly=h * ny, lz=h * nz, radius=3.0 * h, noise=1e-3, seed=nx + nz,
                   **over)
    print(f"[gpu] fused right-hand side {base} {n} {over}", flush=True)
    st = W.droplet_state(cfg)
    ref = S.run(model.Params.from_config(cfg), st, 2)["phi"][0]
    for precision, tol in ((64, 1e-10), (32, 1e-4)):
        g = drpf.Grid(cfg, precision)
        d = g.state(W.droplet_state(cfg))
        g.step(d, 2)
        torch.cuda.synchronize()
        err = np.max(np.abs(d.to_host()["phi"][0] - ref))
        assert err <= tol * np.max(np.abs(ref)), (precision, err)
