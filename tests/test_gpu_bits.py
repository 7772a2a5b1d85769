"""Kernels that stand in for one another round alike, to the last bit of the
state and of the norms (the observables of complex64 states are FP64 sums, in
which another order of the sums or of the layers would show).

The complex64 z pass of a wide contiguous group: alone (its own kernel) and in batches
where another job has a different kind of pass at the same level, so that the
general kernel runs it.  One-workgroup ramps: the norms of renormalized
complex64 ramps as recorded in golden/resident_norms.txt."""
import os

import numpy as np
import pytest
import torch

from paper_2108_13410_amd import workloads, z2h

pytestmark = pytest.mark.gpu

GOLDEN = os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden", "resident_norms.txt")
END = (1.0, 0.9, 0.3, 0.25)


@pytest.mark.parametrize("Lx,Ly", [(3, 4), (2, 6)])
def test_wide_pass_rounds_as_the_general_kernel(Lx, Ly):
    dtype = z2h.Z2H_C64
    M = 3
    print(f"case bits wide {Lx}x{Ly}", flush=True)
    ramp = z2h.schedule(workloads.TORIC, END, M, 0.1, renorm=1)
    plan = z2h.z2h_plan_create(Lx, Ly, dtype)
    psi = z2h.alloc_state(plan)
    ws = z2h.alloc_bytes(z2h.z2h_plan_sizes(plan)["ws_evolve"])
    z2h.z2h_state_init(plan, psi, z2h.Z2H_INIT_PSI1)
    z2h.z2h_evolve(plan, psi, ws, ramp)
    # z-x-z ramps of 1, 2 and 3 steps end in a half pass at the level of the
    # first ramp's z pass of step 1, 2 and 3
    scheds = [ramp] + [z2h.schedule(workloads.TORIC, END, k, 0.1, order=1, renorm=1) for k in (3, 2, 1)]
    b = z2h.z2h_batch_create([Lx] * 4, [Ly] * 4, scheds, [z2h.Z2H_INIT_PSI1] * 4, [END] * 4, dtype)
    states, bws = z2h.alloc_bytes(b.states_bytes), z2h.alloc_bytes(b.ws_bytes)
    obs = torch.zeros((4, z2h.Z2H_OBS_DOUBLES), dtype=torch.float64, device="cuda")
    z2h.z2h_batch_run(b, states, bws, obs)
    off = int(b.offsets[0])
    got = states[off:off + psi.numel() * psi.element_size()].view(psi.dtype)
    assert torch.equal(torch.view_as_real(got), torch.view_as_real(psi))


def resident_norms():
    """Lines 'Lx Ly order: norm of every step' (hexadecimal floats)."""
    out = []
    for Lx, Ly in ((2, 2), (2, 3), (3, 2)):
        for order in (0, 1):
            M = 25
            plan = z2h.z2h_plan_create(Lx, Ly, z2h.Z2H_C64)
            psi = z2h.alloc_state(plan)
            ws = z2h.alloc_bytes(z2h.z2h_plan_sizes(plan)["ws_evolve"])
            norms = torch.zeros(M, dtype=torch.float64, device="cuda")
            z2h.z2h_state_init(plan, psi, z2h.Z2H_INIT_PSI1)
            z2h.z2h_evolve(plan, psi, ws, z2h.schedule(workloads.TORIC, END, M, 0.1, order=order, renorm=1), norms=norms)
            out.append(f"{Lx} {Ly} {order}: " + " ".join(float(x).hex() for x in norms.cpu().numpy()))
    return out


def test_resident_norms_are_the_recorded_ones():
    print("case bits resident", flush=True)
    got, want = resident_norms(), open(GOLDEN).read().split("\n")
    for g, w in zip(got, want):
        assert g == w, np.array([float.fromhex(x) for x in g.split()[3:]])
    assert len(got) == len([w for w in want if w])
