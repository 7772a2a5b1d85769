"""The adjoint's reverse sweep: gradients against central differences of the
oracle on schedules with and without the kernel that holds a state per half
block (one group; groups too large for it; K = 2 and K = 3), and with more
levels than one chunk of tables and partials holds (2x3 complex128: 44)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2108_13410_amd import workloads, z2h

pytestmark = pytest.mark.gpu

CASES = [(2, 2, None, 30), (2, 3, None, 60), (2, 3, "split=6:3:9:0/6:3:9:3", 60), (2, 3, "split=4:2:8:0/4:2:8:4/4:2:8:4", 40),
         (2, 4, None, 40), (2, 4, "split=8:4:11:0/8:4:12:4", 40)]


def loss(Lx, Ly, c1, dt, sZ, sX):
    psi = oracle.init_psi1(Lx, Ly)
    oracle.evolve(Lx, Ly, psi, workloads.TORIC, c1, len(sZ), dt, sZ=sZ, sX=sX)
    o = oracle.observe(Lx, Ly, psi, c1)
    return o["energy"] / o["norm"]


@pytest.mark.parametrize("Lx,Ly,cfg,M", CASES)
def test_gradient_against_differences(Lx, Ly, cfg, M):
    print(f"case adjoint {Lx}x{Ly} {cfg} M={M}", flush=True)
    c1, dt = (1.0, 0.9, 0.3, 0.25), 0.1
    rng = np.random.default_rng(M)
    base = (np.arange(M) + 0.5) / M
    sZ, sX = base + rng.normal(0, 0.01, M), base + rng.normal(0, 0.01, M)
    plan = z2h.z2h_plan_create_config(Lx, Ly, z2h.Z2H_C128, cfg) if cfg else z2h.z2h_plan_create(Lx, Ly, z2h.Z2H_C128)
    sz = z2h.z2h_plan_sizes(plan)
    psi = z2h.alloc_state(plan)
    ws = z2h.alloc_bytes(max(sz["ws_evolve"] + 32 * M + 1024, sz["ws_adjoint"] + 64 * M + 1024))
    sched = z2h.schedule(workloads.TORIC, c1, M, dt, sZ=sZ, sX=sX)
    z2h.z2h_state_init(plan, psi, z2h.Z2H_INIT_PSI1)
    z2h.z2h_evolve(plan, psi, ws, sched)
    g = [torch.full((M,), float("nan"), dtype=torch.float64, device="cuda") for _ in range(2)]
    ws.fill_(0xFF)
    L = z2h.z2h_adjoint(plan, psi, ws, sched, c1, g[0], g[1])
    assert abs(L - loss(Lx, Ly, c1, dt, sZ, sX)) < 1e-10
    gz, gx = g[0].cpu().numpy(), g[1].cpu().numpy()
    h = 1e-5  # central differences: h^2 truncation and 1e-15 / h rounding
    for k in (0, 1, M // 2, M - 1):
        for arr, grad in ((sZ, gz), (sX, gx)):
            d = np.zeros(M)
            d[k] = h
            up = loss(Lx, Ly, c1, dt, sZ + d if arr is sZ else sZ, sX + d if arr is sX else sX)
            dn = loss(Lx, Ly, c1, dt, sZ - d if arr is sZ else sZ, sX - d if arr is sX else sX)
            assert abs((up - dn) / (2 * h) - grad[k]) < 1e-7, (k, arr is sZ)
