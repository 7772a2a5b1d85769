"""The fused gate executors above the small states' pass: tile groups
(fuse = 1) and register groups (fuse = 2) at 23 qubits, the smallest states
they take, on lists with gadgets, runs of CNOTs with and without a control
left over, projections and renormalization, against the oracle's gate-by-gate
application."""
import numpy as np
import pytest
import torch

from test_gpu_fine_gates import gadget_list, oracle_apply

from paper_2108_13410_amd import z2h

pytestmark = pytest.mark.gpu

NQ = 23


@pytest.fixture(scope="module")
def reference():
    rng = np.random.default_rng(NQ)
    gates = gadget_list(NQ, rng, 5)
    psi = rng.normal(size=1 << NQ) + 1j * rng.normal(size=1 << NQ)
    psi /= np.linalg.norm(psi)
    return gates, psi, oracle_apply(NQ, psi, gates)


@pytest.mark.parametrize("fuse", [1, 2])
@pytest.mark.parametrize("dtype", [z2h.Z2H_C128, z2h.Z2H_C64])
def test_executors_against_oracle(reference, dtype, fuse):
    gates, psi, ref = reference
    print(f"case large gates dtype={dtype} fuse={fuse}", flush=True)
    arr = (z2h.z2h_gate * len(gates))(*[z2h.z2h_gate(k, a, b, 0, th) for k, a, b, th in gates])
    ws = z2h.alloc_bytes(z2h.z2h_gates_ws_bytes(NQ))
    st = torch.from_numpy(psi).to(torch.complex128 if dtype == z2h.Z2H_C128 else torch.complex64).cuda()
    z2h.z2h_gates_run(NQ, dtype, st, ws, arr, len(gates), fuse=fuse)
    err = np.abs(st.cpu().numpy().astype(np.complex128) - ref).max()
    # unit norm; each gate rounds an amplitude a few times
    assert err < (1e-15 if dtype == z2h.Z2H_C128 else 6e-7) * len(gates)
