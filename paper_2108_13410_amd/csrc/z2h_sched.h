// Job records, schedule values, phase angles and tables and the level
// sequence on the device, shared by the pass kernels and the one-workgroup
// kernel.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "z2h_internal.h"
#include "z2h_tile.h"

namespace z2h {

// FP64 factors of the phase table live at the start of the exchange
// region: every kernel builds its table while no layout change is in flight
// (before the first exchange of a pass, or after the closing barrier of the
// last one), and the region (at least 2^8 elements) outsizes the factors.
__device__ __forceinline__ double2 *table_scratch(unsigned char *smem) {
    return reinterpret_cast<double2 *>(smem);
}

// Build the phase table T[k][w] = scale * exp(i (alpha (nst - 2k) + beta (n - 2w)))
// in LDS (FP64 angles and products, cast to Real).  Contraction into FMAs is
// off in the schedule, angle and table arithmetic, so every kernel that
// builds a table (in LDS or ahead of time in global memory) rounds the same
// way whatever code surrounds it.  Two stages so that a
// pass can compute the factors while its tile loads are in flight and apply
// the scale (which may depend on a norm reduction) afterwards.
__device__ __forceinline__ void table_factors(double2 *fac, int nst, int n, double alpha, double beta) {
#pragma clang fp contract(off)
    const int t = threadIdx.x, nt = blockDim.x;
    for (int j = t; j < nst + 1 + n + 1; j += nt) {
        double ang = j <= nst ? alpha * (double)(nst - 2 * j) : beta * (double)(n - 2 * (j - nst - 1));
        double s, c;
        sincos(ang, &s, &c);
        fac[j] = make_double2(c, s);
    }
}

template <typename Real>
__device__ __forceinline__ void table_products(Cx<Real> *tab, const double2 *fac, int nst, int n,
                                               double scale) {
#pragma clang fp contract(off)
    const int t = threadIdx.x, nt = blockDim.x;
    __syncthreads();
    const int W = n + 1;
    for (int j = t; j < (nst + 1) * W; j += nt) {
        const int k = j / W, w = j - k * W;
        const double2 a = fac[k], b = fac[nst + 1 + w];
        const double re = (a.x * b.x - a.y * b.y) * scale;
        const double im = (a.x * b.y + a.y * b.x) * scale;
        tab[j] = Cx<Real>{(Real)re, (Real)im};
    }
    __syncthreads();
}

template <typename Real>
__device__ void build_table(Cx<Real> *tab, double2 *fac, int nst, int n, double alpha,
                            double beta, double scale) {
    table_factors(fac, nst, n, alpha, beta);
    table_products<Real>(tab, fac, nst, n, scale);
}

// Multiply every register element by T[k][w]: elements are visited in
// Gray-code order so each step updates the syndrome by one uniform column.
// SPELLED: the product of phase_mul, so that kernels sharing a state round
// alike; else the compiler contracts it as the registers allow.
template <typename Real, int R, int PHASE_CHUNK = 0, bool SPELLED = true>
__device__ __forceinline__ void apply_phase(Cx<Real> (&v)[1 << R], const LayCtx<R> &L, int basis,
                                            int n, const Cx<Real> *tab) {
    uint32_t s = basis ? L.s0x : L.s0z;
    const Cx<Real> *tw = tab + L.w0;
    const int W = n + 1;
#pragma unroll
    for (int idx = 0; idx < (1 << R); ++idx) {
        const int q = idx ^ (idx >> 1);
        if (idx) s ^= basis ? L.lx[__builtin_ctz(idx)] : L.lz[__builtin_ctz(idx)];
        const Cx<Real> f = tw[__umul24((uint32_t)popc(s), (uint32_t)W) + __builtin_popcount(q)];
        v[q] = SPELLED ? phase_mul(v[q], f) : cmul(v[q], f);
        // keep the table reads of at most eight elements in flight (register
        // pressure when a block holds two tiles)
        if (PHASE_CHUNK && (idx & (PHASE_CHUNK - 1)) == PHASE_CHUNK - 1) __builtin_amdgcn_sched_barrier(0);
    }
}

// Sum of |v_q|^2 over a thread's register elements: pairwise in the storage
// precision (complex64 steps accumulate in FP32), returned as FP64 for the
// block and grid reductions.  IM: the form of the squares (abs2).
template <typename Real, int R, bool IM>
__device__ __forceinline__ double sumsq(const Cx<Real> (&v)[1 << R]) {
    Real a[1 << R];
#pragma unroll
    for (int q = 0; q < (1 << R); ++q) a[q] = abs2<IM>(v[q]);
#pragma unroll
    for (int h = (1 << R) >> 1; h > 0; h >>= 1) {
#pragma unroll
        for (int q = 0; q < h; ++q) a[q] += a[q + h];
    }
    return (double)a[0];
}


// Norm partials and traces live in global memory; accessing them through
// global-address-space pointers keeps them off the LDS counter (generic
// "flat" accesses count on both, and would make LDS waits wait for them).
typedef __attribute__((address_space(1))) double *GlobalDoubles;
__device__ __forceinline__ double gld(const double *p, int64_t i) { return ((GlobalDoubles)p)[i]; }
__device__ __forceinline__ void gst(double *p, int64_t i, double v) { ((GlobalDoubles)p)[i] = v; }

// Job records are read-only during a launch: read them through the constant
// address space so that the (block-uniform) record is fetched with scalar
// loads, whose completion does not wait on the block's outstanding tile loads.
typedef const __attribute__((address_space(4))) uint32_t *ConstWords;
static_assert(sizeof(JobDev) % 4 == 0, "job record is copied in 32-bit words");

__device__ __forceinline__ JobDev job_record(const JobDev *jobs, int jb, const JobDev &inl) {
    if (!jobs) return inl;
    JobDev J;
    uint32_t *d = reinterpret_cast<uint32_t *>(&J);
    const ConstWords src = (ConstWords)(jobs + jb);
#pragma unroll
    for (int i = 0; i < (int)(sizeof(JobDev) / 4); ++i) d[i] = src[i];
    return J;
}

// Job of a packed launch's block-job b (index list read through the constant
// address space: a scalar load).
__device__ __forceinline__ int job_index(const int32_t *jidx, int b) {
    typedef const __attribute__((address_space(4))) int32_t *ConstInts;
    return ((ConstInts)jidx)[b];
}

// ---------------------------------------------------------------- schedule

__device__ __forceinline__ double sched_s(const JobDev &J, int k, int zkind) {
#pragma clang fp contract(off)
    typedef const __attribute__((address_space(4))) double *ConstDoubles;
    const double *arr = zkind ? J.sZ : J.sX;
    if (arr) return ((ConstDoubles)arr)[k];  // read-only; scalar load
    return J.sampling ? (double)(k + 1) / (double)J.M : ((double)k + 0.5) / (double)J.M;
}

// (coupling, field) of the given basis at step k: inner (Z) basis uses
// (JB, hz) at sZ, outer (X) basis uses (JA, hx) at sX.
__device__ __forceinline__ void coup(const JobDev &J, int basis, int k, double &Jc, double &h) {
#pragma clang fp contract(off)
    const double s = sched_s(J, k, basis == 0);
    const int ij = basis == 0 ? 1 : 0, ih = basis == 0 ? 3 : 2;
    Jc = (1.0 - s) * J.c0[ij] + s * J.c1[ij];
    h = (1.0 - s) * J.c0[ih] + s * J.c1[ih];
}

// Angles of a phase pass: full step ka (duration dt) or half steps ka, kb.
__device__ __forceinline__ void phase_angles(const JobDev &J, const LevelOp &op, double &alpha,
                                             double &beta) {
#pragma clang fp contract(off)
    double Ja, ha, Jb = 0, hb = 0;
    coup(J, op.basis, op.ka, Ja, ha);
    if (op.full) {
        alpha = J.dt * Ja;
        beta = J.dt * ha;
        return;
    }
    if (op.kb >= 0) coup(J, op.basis, op.kb, Jb, hb);
    alpha = 0.5 * J.dt * (Ja + Jb);
    beta = 0.5 * J.dt * (ha + hb);
}

// Level sequence of one job (see the host planner for the derivation): the
// visited group zig-zags between group 0 (computational basis reached) and
// group K-1 (Hadamard basis reached).
__host__ __device__ inline LevelOp level_op(int lev, int K, int S, int k0, int order) {
    LevelOp op{0, kIdle, 0, -1, -1, 0, 0, 0};
    const int P = 2 * (K - 1);
    const int nlev = order == 0 ? P * (S + 1) + 1 : P * S + 1;
    if (S <= 0 || lev < 0 || lev >= nlev) return op;
    const int r = lev % P;
    op.group = r <= K - 1 ? r : P - r;
    const int j = lev / P;
    if (op.group != 0 && op.group != K - 1) {
        op.kind = kPlainH;
        return op;
    }
    if (op.group == K - 1 && r == K - 1) {
        // outer visit j
        op.basis = 1;
        if (order == 0) {
            op.kind = kPhaseB;
            if (j == 0) {
                op.ka = k0; op.kb = -1; op.full = 0;
            } else if (j == S) {
                op.ka = k0 + S - 1; op.kb = -1; op.full = 0;
            } else {
                op.ka = k0 + j - 1; op.kb = k0 + j; op.full = 0;
            }
            op.renorm = j >= 1 ? 1 : 0;
        } else {
            op.kind = kPhaseB;
            op.ka = k0 + j; op.full = 1;
            op.renorm = 1;
        }
        return op;
    }
    // inner visit j (group 0)
    op.basis = 0;
    if (order == 0) {
        if (j == 0 || j == S + 1) {
            op.kind = kPlainH;
        } else {
            op.kind = kPhaseB;
            op.ka = k0 + j - 1; op.full = 1;
            op.norm = 1;
        }
    } else {
        if (j == 0) {
            op.kind = kHalfIn; op.ka = k0; op.kb = -1; op.full = 0; op.norm = 1;
        } else if (j == S) {
            op.kind = kHalfOut; op.ka = k0 + S - 1; op.kb = -1; op.full = 0;
        } else {
            op.kind = kPhaseB; op.ka = k0 + j - 1; op.kb = k0 + j; op.full = 0; op.norm = 1;
        }
    }
    return op;
}

}  // namespace z2h
