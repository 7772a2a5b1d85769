"""Passes of wide contiguous groups (14 qubits complex64, 13 complex128): the
z passes of a 24-qubit ramp in a kernel of their own, the first and last pass
and the z-x-z order's half passes in the general one.  Against a plan of
narrower groups with another pass order (itself checked against the oracle at
smaller sizes), with norms, renormalization and both step orders, and against
closed forms at zero field."""
import numpy as np
import pytest
import torch

from paper_2108_13410_amd import workloads, z2h

pytestmark = pytest.mark.gpu

WIDE = {z2h.Z2H_C64: "split=14:5:14:0/10:5:14:4", z2h.Z2H_C128: "split=13:4:13:0/11:4:13:2"}
NARROW = "split=8:4:12:0/8:4:12:4/8:4:12:4"


def ramp(dtype, cfg, order, M, c1):
    plan = z2h.z2h_plan_create_config(3, 4, dtype, cfg)
    sz = z2h.z2h_plan_sizes(plan)
    psi = z2h.alloc_state(plan)
    ws = z2h.alloc_bytes(max(sz["ws_evolve"], sz["ws_observe"]))
    norms = torch.zeros(M, dtype=torch.float64, device="cuda")
    z2h.z2h_state_init(plan, psi, z2h.Z2H_INIT_PSI1)
    sched = z2h.schedule(workloads.TORIC, c1, M, 0.1, order=order, renorm=1 if dtype == z2h.Z2H_C64 else 0)
    z2h.z2h_evolve(plan, psi, ws, sched, norms=norms)
    ob = z2h.z2h_observe(plan, psi, ws, c1)
    return psi, norms, ob


@pytest.mark.parametrize("order", [0, 1])
@pytest.mark.parametrize("dtype", [z2h.Z2H_C64, z2h.Z2H_C128])
def test_wide_group_ramp(dtype, order):
    for M in (1, 4):
        print(f"case wide dtype={dtype} order={order} M={M}", flush=True)
        a, na, oa = ramp(dtype, WIDE[dtype], order, M, (1.0, 0.9, 0.3, 0.25))
        b, nb, ob = ramp(dtype, NARROW, order, M, (1.0, 0.9, 0.3, 0.25))
        # each transform layer rounds an amplitude once: 4 x 24 layers a step
        tol = (4e-15 if dtype == z2h.Z2H_C128 else 2e-6) * (M + 1)
        scale = float(b.abs().max())
        assert float((a - b).abs().max()) < tol * scale
        assert float((na - nb).abs().max()) < tol and float((na - 1).abs().max()) < tol
        assert abs(oa["energy"] - ob["energy"]) < 24 * tol


def test_wide_zero_field_phase():
    for dtype in WIDE:
        a, _, _ = ramp(dtype, WIDE[dtype], 0, 6, (1.0, 1.0, 0.0, 0.0))
        plan = z2h.z2h_plan_create_config(3, 4, dtype, WIDE[dtype])
        b = z2h.alloc_state(plan)
        z2h.z2h_state_init(plan, b, z2h.Z2H_INIT_PSI1)
        # stars and plaquettes all +1: the phase exp(i (12 + 12) T)
        ph = complex(np.exp(1j * 24 * 0.6))
        tol = 1e-13 if dtype == z2h.Z2H_C128 else 2e-5
        assert float((a - ph * b).abs().max()) < tol * float(b.abs().max())
