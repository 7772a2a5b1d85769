// The fine tile pass of gate-level circuits on states of at most
// kFineMaxQubits qubits.
//
// The tile pass of larger states has 128 blocks of two waves at 19 qubits,
// and what they wait for is their own code: a gate is one of up to 31
// unrolled variants over 32 amplitudes (185 KB of code in all), fetched cold
// and run once: 36 us a pass, of which its arithmetic is 3 us.  Here a thread
// holds 8 amplitudes, only H, R_x and CNOT targets need their qubit in the
// registers, everything else sees the other bits of the index as constants
// of the thread, and one variant per register bit serves all masks (6 KB of
// code).  15.9 us a pass; with 16 amplitudes a thread 17.1 us (fewer layout
// changes, but more code per gate and half the waves).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/z2h.h"
#include "z2h_gate_tile.h"
#include "z2h_internal.h"
#include "z2h_kernels.h"
#include "z2h_solvers.h"
#include "z2h_tile.h"

namespace z2h {

template <typename Real>
struct FineFile {
    typedef Real type __attribute__((ext_vector_type(2 << kFineBits)));
};
template <typename Real>
using Fine = typename FineFile<Real>::type;

constexpr size_t kFineGateBytes = sizeof(GateDev) * kFuseMaxGates;
static_assert(kFineGateBytes % 16 == 0, "the tile follows the gate records in LDS");

// Parity of register index k under a mask, as a flag of the whole block.
__device__ __forceinline__ bool reg_odd(int k, int mask) { return __builtin_popcount(k & mask) & 1; }

template <typename Real, int B>
__device__ __forceinline__ void fine_pair(Fine<Real> &v, int kind, int mask, const double *m, bool odd) {
    constexpr int N = 1 << kFineBits;
    if (kind == Z2H_GATE_H) {
#pragma unroll
        for (int k = 0; k < N; ++k)
            if (!(k & (1 << B))) {
                const int j = k | (1 << B);
                const Real xr = v[2 * k], xi = v[2 * k + 1], yr = v[2 * j], yi = v[2 * j + 1];
                v[2 * k] = xr + yr;
                v[2 * k + 1] = xi + yi;
                v[2 * j] = xr - yr;
                v[2 * j + 1] = xi - yi;
            }
    } else if (kind == Z2H_GATE_RX) {
        const Real c = (Real)m[0], w = (Real)m[3];
#pragma unroll
        for (int k = 0; k < N; ++k)
            if (!(k & (1 << B))) {
                const int j = k | (1 << B);
                const Real xr = v[2 * k], xi = v[2 * k + 1], yr = v[2 * j], yi = v[2 * j + 1];
                v[2 * k] = c * xr - w * yi;
                v[2 * k + 1] = c * xi + w * yr;
                v[2 * j] = c * yr - w * xi;
                v[2 * j + 1] = c * yi + w * xr;
            }
    } else {
#pragma unroll
        for (int k = 0; k < N; ++k)
            if (!(k & (1 << B))) {
                const int j = k | (1 << B);
                const Real xr = v[2 * k], xi = v[2 * k + 1], yr = v[2 * j], yi = v[2 * j + 1];
                const bool flip = odd != reg_odd(k, mask);
                v[2 * k] = flip ? yr : xr;
                v[2 * k + 1] = flip ? yi : xi;
                v[2 * j] = flip ? xr : yr;
                v[2 * j + 1] = flip ? xi : yi;
            }
    }
}

// g: the gate's record in LDS (the same for the whole block).
template <typename Real>
__device__ __forceinline__ void fine_gate(Fine<Real> &v, const GateDev *g, uint32_t index) {
    static_assert(kFineBits == 3, "the switch below covers three register bits");
    const int kind = __builtin_amdgcn_readfirstlane(g->kind), q0 = __builtin_amdgcn_readfirstlane(g->q0);
    const int q1 = __builtin_amdgcn_readfirstlane(g->q1);
    const bool odd = __builtin_popcount(index & (uint32_t)g->pad) & 1;
    if (kind == Z2H_GATE_RZ) {
        // exp(-+ i theta / 2): the two phases are conjugate
        const Real c = (Real)g->m[0], w = odd ? (Real)g->m[7] : (Real)g->m[1];
#pragma unroll
        for (int k = 0; k < (1 << kFineBits); ++k) {
            const Real wk = reg_odd(k, q0) ? -w : w;
            const Real x = v[2 * k], y = v[2 * k + 1];
            v[2 * k] = c * x - wk * y;
            v[2 * k + 1] = c * y + wk * x;
        }
        return;
    }
    if (kind == Z2H_GATE_PROJ0) {
#pragma unroll
        for (int k = 0; k < (1 << kFineBits); ++k) {
            const bool drop = odd != reg_odd(k, q0);
            v[2 * k] = drop ? (Real)0 : v[2 * k];
            v[2 * k + 1] = drop ? (Real)0 : v[2 * k + 1];
        }
        return;
    }
    switch (kind == Z2H_GATE_CNOT ? q1 : q0) {
        case 0: fine_pair<Real, 0>(v, kind, q0, g->m, odd); break;
        case 1: fine_pair<Real, 1>(v, kind, q0, g->m, odd); break;
        default: fine_pair<Real, 2>(v, kind, q0, g->m, odd); break;
    }
}

// Local index of register 0 of thread t in the layout whose kFineBits bits
// are packed, ascending, in code.
__device__ __forceinline__ uint32_t fine_spread(uint32_t t, uint32_t code) {
    uint32_t x = t;
#pragma unroll
    for (int b = 0; b < kFineBits; ++b) {
        const uint32_t p = (code >> (4 * b)) & 15u;
        x = ((x >> p) << (p + 1)) | (x & ((1u << p) - 1u));
    }
    return x;
}

template <typename Real>
__global__ void __launch_bounds__(1024) fine_kernel(FusedArgs a) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    // the gate records, fetched from the argument block at once (one by one,
    // each would wait for its own cold scalar load)
    GateDev *gates = reinterpret_cast<GateDev *>(smem);
    Cx<Real> *lds = reinterpret_cast<Cx<Real> *>(smem + kFineGateBytes);
    Cx<Real> *st = reinterpret_cast<Cx<Real> *>(a.state);
    const uint32_t t = threadIdx.x, tile = blockIdx.x;
    const int lt = a.m - kFineBits;
    uint32_t home = 0;
#pragma unroll
    for (int b = 0; b < kFineBits; ++b) home |= (uint32_t)(lt + b) << (4 * b);
    const uint64_t base = deposit(t, a.lq, lt) | deposit(tile, a.cq, a.nq - a.m);
    uint64_t off[kFineBits];
#pragma unroll
    for (int b = 0; b < kFineBits; ++b) off[b] = 1ull << a.lq[lt + b];
    Fine<Real> v;
    {
        const uint32_t *src = reinterpret_cast<const uint32_t *>(a.gates);
        for (uint32_t j = t; j < (uint32_t)a.ngates * (uint32_t)(sizeof(GateDev) / 4); j += blockDim.x)
            reinterpret_cast<uint32_t *>(gates)[j] = src[j];
    }
#pragma unroll
    for (int k = 0; k < (1 << kFineBits); ++k) {
        uint64_t i = base;
#pragma unroll
        for (int b = 0; b < kFineBits; ++b)
            if (k & (1 << b)) i |= off[b];
        const Cx<Real> e = st[i];
        v[2 * k] = e.x;
        v[2 * k + 1] = e.y;
    }
    // (register k's slot is the thread's plus the sum of its bits' slots)
    auto move = [&](uint32_t from, uint32_t to) {
        __syncthreads();
#pragma unroll
        for (int side = 0; side < 2; ++side) {
            const uint32_t code = side ? to : from, b0 = lds_slot<Real>(fine_spread(t, code));
            uint32_t so[kFineBits];
#pragma unroll
            for (int b = 0; b < kFineBits; ++b) so[b] = lds_slot<Real>(1u << ((code >> (4 * b)) & 15u));
#pragma unroll
            for (int k = 0; k < (1 << kFineBits); ++k) {
                uint32_t o = b0;
#pragma unroll
                for (int b = 0; b < kFineBits; ++b)
                    if (k & (1 << b)) o += so[b];
                if (side == 0) {
                    lds[o] = Cx<Real>{v[2 * k], v[2 * k + 1]};
                } else {
                    const Cx<Real> e = lds[o];
                    v[2 * k] = e.x;
                    v[2 * k + 1] = e.y;
                }
            }
            if (side == 0) __syncthreads();
        }
    };
    __syncthreads();
    uint32_t cur = home;
    int g = 0;
    for (int p = 0; p < a.nphase; ++p) {
        const uint32_t lay = a.phase[p] & 0xFFFFFu;
        if (lay != cur) {
            move(cur, lay);
            cur = lay;
        }
        const uint32_t index = (tile << a.m) | fine_spread(t, lay);
        for (const int end = (int)(a.phase[p] >> 24); g < end; ++g) fine_gate<Real>(v, gates + g, index);
    }
    if (cur != home) move(cur, home);
    const Real f = (Real)a.scale;
#pragma unroll
    for (int k = 0; k < (1 << kFineBits); ++k) {
        uint64_t i = base;
#pragma unroll
        for (int b = 0; b < kFineBits; ++b)
            if (k & (1 << b)) i |= off[b];
        st[i] = Cx<Real>{v[2 * k] * f, v[2 * k + 1] * f};
    }
}

// Largest padded tile, 2^13 complex64 or 2^12 complex128 amplitudes, and the
// gate records beside it.
constexpr size_t kFineLdsMax = 73728;
static_assert(tile_lds_bytes<float>(13) + kFineGateBytes <= kFineLdsMax &&
                  tile_lds_bytes<double>(12) + kFineGateBytes <= kFineLdsMax, "tile LDS");

hipError_t launch_fine(bool c128, const FusedArgs &a, hipStream_t s) {
    if (a.m < kFineBits || a.m > 13 || a.nq < a.m || a.nq > kFineMaxQubits) return hipErrorInvalidValue;
    const unsigned nb = 1u << (a.nq - a.m), nt = 1u << (a.m - kFineBits);
    const size_t lds = kFineGateBytes + (c128 ? tile_lds_bytes<double>(a.m) : tile_lds_bytes<float>(a.m));
    if (lds > kFineLdsMax || nt > 1024) return hipErrorInvalidValue;
    hipError_t e = set_lds(c128 ? reinterpret_cast<const void *>(&fine_kernel<double>)
                                : reinterpret_cast<const void *>(&fine_kernel<float>), lds);
    if (e != hipSuccess) return e;
    if (c128)
        hipLaunchKernelGGL(fine_kernel<double>, dim3(nb), dim3(nt), lds, s, a);
    else
        hipLaunchKernelGGL(fine_kernel<float>, dim3(nb), dim3(nt), lds, s, a);
    return hipGetLastError();
}

}  // namespace z2h
