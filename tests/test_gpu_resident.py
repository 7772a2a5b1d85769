"""Ramps of the one-workgroup lattices (8 and 12 qubits) against the oracle:
step counts around the chunks the phase tables are built in (12 phases, two a
step), both step orders, per-step norms and renormalization."""
import numpy as np
import pytest

from helpers import (compare_observables, fidelity_loss, gpu_run, oracle_observables, oracle_run, to_oracle_order)
from paper_2108_13410_amd import workloads, z2h

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("order", [0, 1])
@pytest.mark.parametrize("dtype", [z2h.Z2H_C128, z2h.Z2H_C64])
@pytest.mark.parametrize("Lx,Ly", [(2, 2), (2, 3), (3, 2)])
def test_resident_ramp(Lx, Ly, dtype, order):
    n, c1 = 2 * Lx * Ly, (1.0, 0.9, 0.35, 0.2)
    for M in (1, 5, 6, 12, 40):
        renorm = 1 if dtype == z2h.Z2H_C64 else 0
        print(f"case resident {Lx}x{Ly} dtype={dtype} order={order} M={M}", flush=True)
        g, ob, norms = gpu_run(Lx, Ly, dtype, workloads.TORIC, c1, M, 0.1, order=order, renorm=renorm)
        o = oracle_run(Lx, Ly, workloads.TORIC, c1, M, 0.1, order=order)
        tol = 1e-12 if dtype == z2h.Z2H_C128 else 1e-5
        assert fidelity_loss(o, to_oracle_order(Lx, Ly, g)) < tol
        assert np.abs(norms - 1.0).max() < tol
        compare_observables(ob, oracle_observables(Lx, Ly, o, c1), 1e-10 if dtype == z2h.Z2H_C128 else 1e-5, n)
