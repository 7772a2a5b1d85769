// Butterflies across the lanes of a wave, without LDS.
//
// A lane stands for the logical index wave_lane(l): the directions of its
// six bits are the lane exchanges that cost one instruction, xor 1 and 2
// (quad permutes), 7 (half-row mirror), 8 (row rotation), 16 and 32 (row and
// half-wave swaps).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "z2h_tile.h"

namespace z2h {

// Logical index of lane l: flipping logical bit b is the lane exchange of
// direction b above.
__device__ __forceinline__ uint32_t wave_lane(uint32_t l) { return l ^ ((l & 4u) ? 3u : 0u); }

template <int B>
__device__ __forceinline__ int dpp32(int x) {
    static_assert(B >= 0 && B < 4, "directions within a row of 16 lanes");
    constexpr int ctrl = B == 0 ? 0xB1 : B == 1 ? 0x4E : B == 2 ? 0x141 : 0x128;
    return __builtin_amdgcn_update_dpp(0, x, ctrl, 0xf, 0xf, true);
}

// x of the lane across direction B (B < 4).
template <int B>
__device__ __forceinline__ float lane_across(float x) {
    return __builtin_bit_cast(float, dpp32<B>(__builtin_bit_cast(int, x)));
}
template <int B>
__device__ __forceinline__ double lane_across(double x) {
    const uint64_t u = __builtin_bit_cast(uint64_t, x);
    const uint32_t lo = (uint32_t)dpp32<B>((int)(uint32_t)u), hi = (uint32_t)dpp32<B>((int)(uint32_t)(u >> 32));
    return __builtin_bit_cast(double, (uint64_t)lo | ((uint64_t)hi << 32));
}

// Exchange of the lane bit of direction B (4 or 5) with the register bit
// that tells a from b: a keeps its lower lanes and takes b's, b the upper.
template <int B>
__device__ __forceinline__ void swap32(uint32_t &a, uint32_t &b) {
    static_assert(B == 4 || B == 5, "rows or halves of a wave");
    if constexpr (B == 4) {
        const auto r = __builtin_amdgcn_permlane16_swap(a, b, false, false);
        a = r[0];
        b = r[1];
    } else {
        const auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
        a = r[0];
        b = r[1];
    }
}
template <int B>
__device__ __forceinline__ void lane_swap(float &a, float &b) {
    uint32_t x = __builtin_bit_cast(uint32_t, a), y = __builtin_bit_cast(uint32_t, b);
    swap32<B>(x, y);
    a = __builtin_bit_cast(float, x);
    b = __builtin_bit_cast(float, y);
}
template <int B>
__device__ __forceinline__ void lane_swap(double &a, double &b) {
    const uint64_t u = __builtin_bit_cast(uint64_t, a), v = __builtin_bit_cast(uint64_t, b);
    uint32_t xl = (uint32_t)u, xh = (uint32_t)(u >> 32), yl = (uint32_t)v, yh = (uint32_t)(v >> 32);
    swap32<B>(xl, yl);
    swap32<B>(xh, yh);
    a = __builtin_bit_cast(double, (uint64_t)xl | ((uint64_t)xh << 32));
    b = __builtin_bit_cast(double, (uint64_t)yl | ((uint64_t)yh << 32));
}

// a, b, c, d += s times the value of the lane across direction B, each in one
// instruction (the compiler makes a move and a multiply-add of it).  The
// leading wait covers a register that the instruction before has written.
template <int B>
__device__ __forceinline__ void fmac4_across(float &a, float &b, float &c, float &d, float s) {
#define Z2H_FMAC4(CTRL)                                                          \
    asm("s_nop 1\n\t"                                                            \
        "v_fmac_f32_dpp %0, %0, %4 " CTRL " row_mask:0xf bank_mask:0xf\n\t"      \
        "v_fmac_f32_dpp %1, %1, %4 " CTRL " row_mask:0xf bank_mask:0xf\n\t"      \
        "v_fmac_f32_dpp %2, %2, %4 " CTRL " row_mask:0xf bank_mask:0xf\n\t"      \
        "v_fmac_f32_dpp %3, %3, %4 " CTRL " row_mask:0xf bank_mask:0xf"           \
        : "+v"(a), "+v"(b), "+v"(c), "+v"(d)                                      \
        : "v"(s))
    if constexpr (B == 0) Z2H_FMAC4("quad_perm:[1,0,3,2]");
    else if constexpr (B == 1) Z2H_FMAC4("quad_perm:[2,3,0,1]");
    else if constexpr (B == 2) Z2H_FMAC4("row_half_mirror");
    else Z2H_FMAC4("row_ror:8");
#undef Z2H_FMAC4
}

// One butterfly layer along lane direction B of every register element;
// directions 5 and 4 trade places with register bit T.
//
// Within a row the partner's value comes with the multiply-add itself: a
// lane forms own + s other with s = -1 in the upper lanes, which leaves the
// upper lane's difference negated.  A transform that ends in a diagonal and
// its way back meet that sign twice: FWD leaves it, !FWD takes a vector that
// carries it (s = +1 in the upper lanes).  Every product with s is exact, so
// the sums are those of the plain butterfly.
template <int B, bool FWD, int T = 0, typename Real, int N>
__device__ __forceinline__ void lane_layer(Cx<Real> (&v)[N], uint32_t lam) {
    if constexpr (B < 4) {
        const Real s = (((lam >> B) & 1u) != 0) == FWD ? (Real)-1 : (Real)1;
        if constexpr (sizeof(Real) == 4) {
#pragma unroll
            for (int q = 0; q < N; q += 2) fmac4_across<B>(v[q].x, v[q].y, v[q + 1].x, v[q + 1].y, s);
        } else {
#pragma unroll
            for (int q = 0; q < N; ++q) {
                v[q].x = __builtin_fma(s, lane_across<B>(v[q].x), v[q].x);
                v[q].y = __builtin_fma(s, lane_across<B>(v[q].y), v[q].y);
            }
        }
    } else {
        constexpr int r = 1 << T;
        static_assert(N > r, "the register bit that trades places");
        auto swap = [&]() {
#pragma unroll
            for (int q = 0; q < N; ++q)
                if (!(q & r)) {
                    lane_swap<B>(v[q].x, v[q | r].x);
                    lane_swap<B>(v[q].y, v[q | r].y);
                }
        };
        if constexpr (FWD) swap();
#pragma unroll
        for (int q = 0; q < N; ++q)
            if (!(q & r)) {
                const Cx<Real> a = v[q], b = v[q | r];
                v[q] = cadd(a, b);
                v[q | r] = csub(a, b);
            }
        if constexpr (!FWD) swap();
    }
}

// Directions [LO, HI) below 4, lowest first.
template <int LO, int HI, bool FWD, typename Real, int N>
__device__ __forceinline__ void row_layers(Cx<Real> (&v)[N], uint32_t lam) {
    if constexpr (LO < HI) {
        lane_layer<LO, FWD>(v, lam);
        row_layers<LO + 1, HI, FWD>(v, lam);
    }
}

// Wave sum, every lane, over the logical lane bits from the highest down.
__device__ __forceinline__ double wave_sum_lanes(double x) {
    double y = x;
    lane_swap<5>(x, y);
    x += y;
    y = x;
    lane_swap<4>(x, y);
    x += y;
    x += lane_across<3>(x);
    x += lane_across<2>(x);
    x += lane_across<1>(x);
    return x + lane_across<0>(x);
}

// Butterflies over register bits [lo, hi).
template <int LO, int HI, typename Real, int N>
__device__ __forceinline__ void reg_layers(Cx<Real> (&v)[N]) {
#pragma unroll
    for (int j = LO; j < HI; ++j)
#pragma unroll
        for (int q = 0; q < N; ++q)
            if (!(q & (1 << j))) {
                const Cx<Real> a = v[q], b = v[q | (1 << j)];
                v[q] = cadd(a, b);
                v[q | (1 << j)] = csub(a, b);
            }
}

// Exchange of the wave bits with the high WB register bits, through buf.
// CX: the real, then the imaginary parts, through half the LDS; buf may then
// be used again after the call without a barrier (else after the next one).
template <int RB, int WB, bool CX, typename Real>
__device__ __forceinline__ void wave_exchange(Cx<Real> (&v)[1 << RB], Cx<Real> *buf, uint32_t wave, uint32_t lane) {
    constexpr int keep = RB - WB;
    constexpr uint32_t km = (1u << keep) - 1u;
    auto to = [&](uint32_t q) { return (((wave << RB) | q) << 6) | lane; };
    auto from = [&](uint32_t q) { return ((((q >> keep) << RB) | (wave << keep) | (q & km)) << 6) | lane; };
    if constexpr (CX) {
        Real *b = reinterpret_cast<Real *>(buf);
#pragma unroll
        for (uint32_t q = 0; q < (1u << RB); ++q) b[to(q)] = v[q].x;
        __syncthreads();
#pragma unroll
        for (uint32_t q = 0; q < (1u << RB); ++q) v[q].x = b[from(q)];
        __syncthreads();
#pragma unroll
        for (uint32_t q = 0; q < (1u << RB); ++q) b[to(q)] = v[q].y;
        __syncthreads();
#pragma unroll
        for (uint32_t q = 0; q < (1u << RB); ++q) v[q].y = b[from(q)];
        __syncthreads();
    } else {
#pragma unroll
        for (uint32_t q = 0; q < (1u << RB); ++q) buf[to(q)] = v[q];
        __syncthreads();
#pragma unroll
        for (uint32_t q = 0; q < (1u << RB); ++q) v[q] = buf[from(q)];
    }
}

// Transform of a tile of RB + 6 + WB qubits held with lane bits 0-5, wave
// bits above and register bits on top; it ends in the layout of wave_index.
// bwd_wave transforms from that layout and ends in the first one.  The C
// lowest qubits are carried along, not transformed.
template <int RB, int WB, bool CX, int C = 0, typename Real>
__device__ __forceinline__ void fwd_wave(Cx<Real> (&v)[1 << RB], Cx<Real> *buf, uint32_t wave, uint32_t lane, uint32_t lam) {
    static_assert(C <= 4, "carried qubits are lanes of a row");
    reg_layers<0, RB>(v);
    lane_layer<4, true, 0>(v, lam);
    lane_layer<5, true, 1>(v, lam);
    if constexpr (WB != 0) {
        wave_exchange<RB, WB, CX>(v, buf, wave, lane);
        reg_layers<RB - WB, RB>(v);
        row_layers<C, 4, true>(v, lam);
    } else {
        row_layers<(C < 2 ? 2 : C), 4, true>(v, lam);
        row_layers<(C < 2 ? C : 2), 2, true>(v, lam);
    }
}

template <int RB, int WB, bool CX, int C = 0, typename Real>
__device__ __forceinline__ void bwd_wave(Cx<Real> (&v)[1 << RB], Cx<Real> *buf, uint32_t wave, uint32_t lane, uint32_t lam) {
    // (the register bits that lane bits 4 and 5 trade places with may sit in
    // wave bits until the exchange back)
    constexpr bool early4 = WB == 0 || RB - WB >= 1, early5 = WB == 0 || RB - WB >= 2;
    row_layers<C, 4, false>(v, lam);
    if constexpr (early4) lane_layer<4, false, 0>(v, lam);
    if constexpr (early5) lane_layer<5, false, 1>(v, lam);
    if constexpr (WB != 0) {
        reg_layers<RB - WB, RB>(v);
        wave_exchange<RB, WB, CX>(v, buf, wave, lane);
    }
    if constexpr (!early4) lane_layer<4, false, 0>(v, lam);
    if constexpr (!early5) lane_layer<5, false, 1>(v, lam);
    reg_layers<0, RB>(v);
}

// Index of register element q of a thread after fwd_wave.
template <int RB, int WB>
__device__ __host__ constexpr uint32_t wave_index(uint32_t wave, uint32_t lam, uint32_t q) {
    constexpr int keep = RB - WB;
    const uint32_t w = WB ? q >> keep : 0u;                                   // wave bits, in the registers
    const uint32_t e = WB ? (wave << keep) | (q & ((1u << keep) - 1u)) : q;   // element before the exchange
    // before it, lane bits 4 and 5 traded places with element bits 0 and 1
    const uint32_t lo = (lam & 15u) | ((e & 1u) << 4) | ((e & 2u) << 4);
    const uint32_t el = (e & ~3u) | ((lam >> 4) & 3u);
    return lo | (w << 6) | (el << (6 + WB));
}

// Tile index bit of register bit r after fwd_wave.
template <int RB, int WB>
constexpr int wave_reg_bit(int r) {
    return WB && r >= RB - WB ? 6 + (r - (RB - WB)) : r < 2 ? 4 + r : 6 + WB + r;
}

}  // namespace z2h
