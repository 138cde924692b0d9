"""Steps whose polymer update runs on a stream of the library's own: one call of several steps gives the
bits of as many calls of one step, whose update stays on the caller's stream: two calls in a row, on
another stream and on the default one, with the finite check in between."""
from __future__ import annotations

import pytest

import workloads as W

pytestmark = pytest.mark.gpu

GRIDS = {"3d": dict(nx=64, ny=32, nz=32), "2d": dict(nx=64, ny=1, nz=32)}


@pytest.mark.parametrize("precision", [64, 32])
@pytest.mark.parametrize("over", [{"advection": 1}, {"advection": 1, "giesekus_alpha": 0.2}, {"constitutive": 1}],
                         ids=["weno", "weno-giesekus", "lcr"])
@pytest.mark.parametrize("dim", list(GRIDS))
def test_steps_of_one_call(dim, over, precision):
    import torch
    import paper_2111_04577_amd as drpf
    n = GRIDS[dim]
    cfg = W.config("C3", **n, lx=1.0, ly=n["ny"] / 64.0, lz=0.5, radius=0.2, noise=1e-3, seed=8, check_finite_every=3,
                   **over)
    print(f"[gpu] steps of one call {dim} {over} FP{precision}", flush=True)
    g, other = drpf.Grid(cfg, precision), drpf.Grid(cfg, precision)
    a, b = g.state(W.droplet_state(cfg)), other.state(W.droplet_state(cfg))
    for _ in range(10):
        other.step(b, 1)
    torch.cuda.synchronize()
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    g.step(a, 5, stream=s)
    torch.cuda.current_stream().wait_stream(s)
    g.step(a, 5)
    torch.cuda.synchronize()
    for x, y in zip([*a.phi, *a.u, *a.v, *a.w, *a.p, *a.tau[0], *a.tau[1]],
                    [*b.phi, *b.u, *b.v, *b.w, *b.p, *b.tau[0], *b.tau[1]]):
        assert torch.equal(x, y)
