"""Batches of one-workgroup ramps (12 qubits) with more states than CUs: the
same results as one by one, and two states share a CU."""
import time

import numpy as np
import pytest
import torch

from paper_2108_13410_amd import workloads, z2h

pytestmark = pytest.mark.gpu


class Batch:
    def __init__(self, count, dtype, order, M):
        rng = np.random.default_rng(5)
        self.ends = [(1.0, 1.0, *rng.uniform(0, 0.6, 2)) for _ in range(count)]
        self.steps = [M] * count
        renorm = 1 if dtype == z2h.Z2H_C64 else 0
        self.scheds = [z2h.schedule(workloads.TORIC, e, M, 0.1, order=order, renorm=renorm) for e in self.ends]
        self.b = z2h.z2h_batch_create([2] * count, [3] * count, self.scheds, [z2h.Z2H_INIT_PSI1] * count, self.ends, dtype)
        self.states = z2h.alloc_bytes(self.b.states_bytes)
        self.ws = z2h.alloc_bytes(self.b.ws_bytes)
        self.obs = torch.zeros((count, z2h.Z2H_OBS_DOUBLES), dtype=torch.float64, device="cuda")

    def run(self):
        z2h.z2h_batch_run(self.b, self.states, self.ws, self.obs)
        torch.cuda.synchronize()


@pytest.mark.parametrize("order", [0, 1])
@pytest.mark.parametrize("dtype", [z2h.Z2H_C64, z2h.Z2H_C128])
def test_more_states_than_cus(dtype, order):
    """Steps around the phases a kernel builds tables for at once (11)."""
    n, psi = 12, None
    for M in (1, 5, 6, 17):
        print(f"case resident batch dtype={dtype} order={order} M={M}", flush=True)
        big = Batch(300, dtype, order, M)
        big.run()
        plan = z2h.z2h_plan_create(2, 3, dtype)
        ws = z2h.alloc_bytes(max(z2h.z2h_plan_sizes(plan)["ws_evolve"], z2h.z2h_plan_sizes(plan)["ws_observe"]))
        raw = big.states.cpu().numpy()
        for j in (0, 255, 256, 299):
            psi = z2h.alloc_state(plan)
            z2h.z2h_state_init(plan, psi, z2h.Z2H_INIT_PSI1)
            z2h.z2h_evolve(plan, psi, ws, big.scheds[j])
            one = psi.cpu().numpy()
            off = int(big.b.offsets[j])
            assert np.array_equal(raw[off:off + one.nbytes].view(one.dtype), one), (M, j)
    assert psi.numel() == 1 << n


@pytest.mark.parametrize("order", [0, 1])
def test_states_share_cus(order):
    """4096 complex64 states against 256, one a CU: 14 times as long where
    every further 256 wait for the ones before, 9 where two run side by side
    (complex128: 14 and 12, too near for a bound; its registers and LDS are
    checked where they are laid out)."""
    t = []
    for count in (256, 4096):
        b = Batch(count, z2h.Z2H_C64, order, 100)
        b.run()
        best = 1e9
        for _ in range(9):
            t0 = time.perf_counter()
            b.run()
            best = min(best, time.perf_counter() - t0)
        t.append(best)
        print(f"case resident share order={order} count={count}: {best * 1e6:.0f} us", flush=True)
    assert t[1] < 11.5 * t[0]
