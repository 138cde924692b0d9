"""GPU parity of the standalone solve at the edges of its wall-normal transform: the shallowest
and deepest columns, one-line tiles, 2D grids, every wall kind with wall data, both precisions.
FP64 against the oracle's exact solve: 1e-12 of the largest entry (transforms and quotients of
order log2(n) round-offs). FP32 grids transform in x and y in FP32 and solve across the walls in
FP64: storage and transform round-off, 32 eps = 4e-6 (entries of order one, well-conditioned
shift)."""
from __future__ import annotations

import numpy as np
import pytest

import workloads as W
from oracle import discrete as D
from oracle import model

pytestmark = pytest.mark.gpu

KIND = {"neumann": "neumann", "dirichlet": "dirichlet", "face_dirichlet": "wface"}
GRIDS = [("fine", 4, 4, 4), ("coarse", 4, 1, 4), ("coarse", 8, 4, 16), ("fine", 32, 1, 64), ("coarse", 64, 16, 128),
         ("fine", 4, 1, 512)]


@pytest.mark.parametrize("bc", list(KIND))
@pytest.mark.parametrize("which,nx,ny,nz", GRIDS)
def test_solve_sizes(which, nx, ny, nz, bc):
    import torch
    import paper_2111_04577_amd as drpf
    cfg = W.config("C1", nx=nx, ny=ny, nz=nz, lx=1.0, ly=0.7, lz=1.3)
    P = model.Params.from_config(cfg)
    h = P.hf if which == "fine" else P.h
    print(f"[gpu] solve {which} {nx}x{ny}x{nz} {bc}", flush=True)
    for precision, tol in ((64, 1e-12), (32, 4e-6)):
        g = drpf.Grid(cfg, precision)
        shape = g.fine_shape if which == "fine" else g.coarse_shape
        rng = np.random.default_rng(nz)
        dt = g.torch_dtype
        rhs = torch.tensor(rng.standard_normal(shape), dtype=dt)
        wall = torch.tensor(1e-3 * rng.standard_normal((2,) + shape[1:]), dtype=dt)
        shifts = [(0.8, 900.0)] + ([(1.0, 0.0)] if bc == "neumann" and precision == 64 else [])
        for coeff, shift in shifts:
            for walls in (None, wall):
                x = g.helmholtz_solve(rhs.cuda(), which, bc, coeff, shift,
                                      wall=None if walls is None else walls.cuda())
                torch.cuda.synchronize()
                r = rhs.double().numpy().copy()
                if bc == "face_dirichlet":
                    r[-1] = 0.0
                ws = None if walls is None else tuple(walls.double().numpy())
                ref = D.helmholtz(r, coeff, shift, KIND[bc], h, ws)
                err = np.max(np.abs(x.double().cpu().numpy() - ref))
                assert err <= tol * np.max(np.abs(ref)), (precision, shift, walls is None, err, np.max(np.abs(ref)))
