// Index and LDS helpers shared by the gate-level tile passes.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "z2h_tile.h"

namespace z2h {

// The bits of x deposited, lowest first, at the qubits q[0..n).
__device__ __forceinline__ uint64_t deposit(uint64_t x, const int32_t *q, int n) {
    uint64_t g = 0;
    for (int j = 0; j < n; ++j) g |= ((x >> j) & 1ull) << q[j];
    return g;
}

// LDS slot of local index i: one pad element after every 256-byte row, so
// threads whose indices differ only in higher bits reach different banks.
// For indices with disjoint bits the slot is additive, slot(a | b) =
// slot(a) + slot(b) (the low parts of a and b add without a carry), so a
// register's slot is the thread's slot plus a block-uniform offset.
template <typename Real>
constexpr int kPadShift = sizeof(Real) == 8 ? 4 : 5;

template <typename Real>
__device__ __forceinline__ uint32_t lds_slot(uint32_t i) {
    return i + (i >> kPadShift<Real>);
}

template <typename Real>
constexpr size_t tile_lds_bytes(int m) {
    return (((size_t)1 << m) + ((size_t)1 << m >> kPadShift<Real>)) * sizeof(Cx<Real>);
}

}  // namespace z2h
