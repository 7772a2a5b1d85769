"""The Hamiltonian's passes over complex128 states of 16, 18, 20 and 24 qubits
(two groups of qubits whatever the plan's) through the Lanczos entry points: the recurrence's
coefficients against the recurrence written out with H x and inner products
(H x itself is checked against the oracle's rows), the Ritz vector against the
sum of those vectors, for even and odd iteration counts and plans with other
groups."""
import numpy as np
import pytest
import torch

from paper_2108_13410_amd import z2h

pytestmark = pytest.mark.gpu


def start(n):
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    return torch.randn(1 << n, dtype=torch.complex128, device="cuda", generator=g)


@pytest.mark.parametrize("Lx,Ly,cfg,iters", [(3, 4, None, 2), (3, 4, "split=8:4:12:0/8:4:12:4/8:4:12:4", 5), (6, 2, None, 6),
                                             (2, 4, None, 1), (4, 2, None, 6), (3, 3, None, 7), (2, 5, None, 6), (5, 2, None, 3)])
def test_lanczos_two_groups(Lx, Ly, cfg, iters):
    print(f"case lanczos {Lx}x{Ly} {cfg} iters={iters}", flush=True)
    plan = z2h.z2h_plan_create_config(Lx, Ly, z2h.Z2H_C128, cfg) if cfg else z2h.z2h_plan_create(Lx, Ly, z2h.Z2H_C128)
    H = (1.0, 0.8, 0.5, 0.3)
    n = 2 * Lx * Ly
    v = start(n)
    ws = z2h.alloc_bytes(z2h.z2h_lanczos_sizes(plan, iters))
    _, its, alpha, beta = z2h.z2h_lanczos_ground(plan, v, ws, H, max_iter=iters, tol=0.0)
    assert its == iters
    v = start(n)
    energy, residual = z2h.z2h_lanczos_vector(plan, v, H, alpha, beta)

    u = start(n)
    q = [u / torch.linalg.vector_norm(u)]
    y = torch.empty_like(u)
    ra, rb = [], []
    for k in range(iters):
        z2h.z2h_hamiltonian_apply(plan, q[k], y, H)
        a = float(torch.sum((q[k].conj() * y).real))
        r = y - a * q[k] - (rb[-1] * q[k - 1] if k else 0)
        ra.append(a)
        rb.append(float(torch.linalg.vector_norm(r)))
        q.append(r / rb[-1])
    # 2 x 24 transform layers round once each, sums of 2^24 terms in any
    # order stay within sqrt(2^24) eps of their scale, |H| < 60; each
    # iteration amplifies the one before by no more than |H| / beta < 20
    tol = 60 * 48 * 2.3e-16 * 20
    assert np.allclose(alpha, ra, rtol=0, atol=tol) and np.allclose(beta[:iters - 1], rb[:iters - 1], rtol=0, atol=tol)
    T = np.diag(ra) + np.diag(rb[:iters - 1], 1) + np.diag(rb[:iters - 1], -1)
    w, V = np.linalg.eigh(T)
    ref = sum(float(V[k, 0]) * q[k] for k in range(iters))
    ref /= torch.linalg.vector_norm(ref)
    overlap = abs(complex(torch.sum(ref.conj() * v)))
    assert abs(overlap - 1) < tol and abs(energy - w[0]) < 10 * tol
    assert abs(residual - rb[iters - 1] * abs(V[iters - 1, 0])) < 10 * tol
