"""GPU parity of the log-conformation update at the ends of the range of Theta: zero and tiny
entries, equal and nearly equal eigenvalues, entries whose squares underflow, and stretches of
e^12. One step against the FP64 oracle from the same state; 1e-10 of the largest entry of the
family (the update is a few hundred FP64 operations per cell on eigenvalues of that size; the
eigensolve's own error is 1e-15 of the largest eigenvalue)."""
from __future__ import annotations

import numpy as np
import pytest

import workloads as W
from oracle import model
from oracle import step as S

pytestmark = pytest.mark.gpu

CFG = W.config("C3", nx=16, ny=8, nz=8, lx=1.0, ly=0.5, lz=0.5, radius=0.2, noise=1e-3, seed=9, wi=0.5,
               constitutive=1)


def theta_of(kind, shape):
    n = int(np.prod(shape))
    r = 2.0 * W.splitmix64_uniform(3, 6 * n) - 1.0
    rnd = [r[m * n:(m + 1) * n].reshape(shape) for m in range(6)]
    one, zero = np.ones(shape), np.zeros(shape)
    if kind == "zero":
        return [zero.copy() for _ in range(6)]
    if kind == "tiny":
        return [1e-12 * a for a in rnd]
    if kind == "underflow":  # one off-diagonal whose square leaves the range beside ordinary entries
        return [rnd[0], rnd[1], rnd[2], 1e-170 * rnd[3], 1e-141 * rnd[4], zero.copy()]
    if kind == "equal":  # two equal eigenvalues, and all three, in rotated frames
        v = np.stack([rnd[0], rnd[1], rnd[2]]) / np.sqrt(sum(a * a for a in rnd[:3]))
        s = np.where(rnd[3] > 0.0, 0.7, 1e-9)
        return [0.3 * one + s * v[0] * v[0], 0.3 * one + s * v[1] * v[1], 0.3 * one + s * v[2] * v[2],
                s * v[0] * v[1], s * v[0] * v[2], s * v[1] * v[2]]
    if kind == "stretched":
        return [12.0 * one + rnd[0], 11.0 * one, 12.0 * one, rnd[3], rnd[4], rnd[5]]
    raise ValueError(kind)


@pytest.mark.parametrize("kind,alpha", [("zero", 0.2), ("tiny", 0.0), ("underflow", 0.2), ("equal", 0.2),
                                        ("stretched", 0.0)])
def test_theta_range(kind, alpha):
    import torch
    import paper_2111_04577_amd as drpf
    cfg = CFG.replace(giesekus_alpha=alpha)
    print(f"[gpu] log-conformation range {kind}", flush=True)
    st = W.droplet_state(cfg)
    st["theta"] = theta_of(kind, W.coarse_shape(cfg))
    g = drpf.Grid(cfg, 64)
    d = g.state({**st, "theta": [a.copy() for a in st["theta"]]})
    g.step(d, 1)
    torch.cuda.synchronize()
    out = d.to_host()
    ref = S.run(model.Params.from_config(cfg), st, 1)
    for key, got, want in (("theta", out["theta"], ref["theta"]), ("tau", out["tau"][0], ref["tau"][0])):
        big = max(float(np.max(np.abs(a))) for a in want)
        err = max(float(np.max(np.abs(a - b))) for a, b in zip(got, want))
        assert err <= 1e-10 * big, (kind, key, err, big)
