"""GPU parity of the marching passes where a block marches several layers: the fused Cahn-Hilliard
right-hand side and x transform (the hand-over of its two layer slots and of the coarse velocities, the
batches of four layers) and the single-resolution restricted set (its layer rings). A block marches
layers / (resident blocks per column) of them, so this takes many columns: a small periodic problem
repeated along y (2D: x), whose solution is the small one's repeated, against the FP64 oracle on the small
one. In FP64 every case that takes a march asks for two to sixteen times the threads that the card holds
at once. Two steps
(start-up and BDF2): FP64 1e-10 of the largest entry (round-off of a stiff solve, as in every parity
test here), FP32 phi 1e-4 (its 1e-6 of the fourth-order right-hand side over two steps)."""
from __future__ import annotations

import numpy as np
import pytest

import workloads as W
from oracle import model
from oracle import step as S

pytestmark = pytest.mark.gpu

RELAX = {"d_w": 0.1}
WENO = {"advection": 1}
SINGLE = {"refine": 1}
MOVE = {"u_wall_bottom": (0.3, -0.1), "u_wall_top": (-0.2, 0.4)}
# phase-field points (nx, ny, nz) of the small problem, repeats along y (2D: along x), options
CASES = [
    ((128, 8, 64), 128, {}),
    ((128, 8, 64), 128, RELAX),
    ((128, 8, 64), 128, WENO),
    ((128, 8, 64), 128, MOVE),
    ((128, 8, 64), 128, {**SINGLE, **RELAX}),
    ((128, 8, 64), 128, {**SINGLE, **WENO}),
    ((128, 8, 64), 32, {**WENO, **RELAX}),
    ((128, 8, 32), 128, {**SINGLE}),
    ((512, 8, 32), 16, RELAX),             # the widest FP64 rows: two of them and 85 KB of LDS per block
    ((1024, 8, 16), 32, RELAX),            # the widest FP32 rows
    ((64, 1, 1024), 16, {}),               # 2D: one row per block, two layers
    ((32, 1, 1024), 32, RELAX),
]


@pytest.mark.parametrize("n,reps,over", CASES, ids=[f"{c[0]}x{c[1]}-" + "-".join(c[2]) for c in CASES])
def test_marches_of_several_layers(n, reps, over):
    import torch
    import paper_2111_04577_amd as drpf
    r = over.get("refine", 2)
    two_d = n[1] == 1
    nx, ny, nz = n[0] // r, 1 if two_d else n[1] // r, n[2] // r
    h = 1.0 / 16
    small = W.config("C1" if two_d else "C2", nx=nx, ny=ny, nz=nz, lx=h * nx, ly=h * ny, lz=h * nz, radius=3.0 * h,
                     noise=1e-3, seed=nx + nz, rho_ratio=10.0, mu_ratio=5.0, theta_bottom_deg=60.0, **over)
    axis = 2 if two_d else 1
    big = small.replace(nx=nx * reps, lx=small.lx * reps) if two_d else small.replace(ny=ny * reps, ly=small.ly * reps)
    print(f"[gpu] march of several layers {n} repeated {reps} times {over}", flush=True)
    rep = lambda a: np.repeat(np.expand_dims(a, axis), reps, axis).reshape(
        [s * (reps if d == axis else 1) for d, s in enumerate(a.shape)])
    st = W.droplet_state(small)
    ref = S.run(model.Params.from_config(small), st, 2)
    print("[gpu] oracle done", flush=True)
    vmax = max(float(np.max(np.abs(ref[k][0]))) for k in "uvw")
    for precision in (64, 32):
        g = drpf.Grid(big, precision)
        d = g.state({k: [rep(a) for a in v] if k in ("phi", "u", "v", "w", "p") else v for k, v in st.items()})
        g.step(d, 2)
        torch.cuda.synchronize()
        for k in ("phi",) if precision == 32 else ("phi", "u", "v", "w"):
            out = getattr(d, k)[0].double().cpu().numpy()
            den = float(np.max(np.abs(ref[k][0]))) if k == "phi" else vmax
            err = max(float(np.max(np.abs(o - ref[k][0]))) for o in np.split(out, reps, axis))
            print(f"[gpu] FP{precision} {k}: {err / den:.2e}", flush=True)
            assert err <= (1e-4 if precision == 32 else 1e-10) * den, (precision, k, err, den)
        del g, d
        torch.cuda.empty_cache()
