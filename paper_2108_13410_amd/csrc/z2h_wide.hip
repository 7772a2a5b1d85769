// Pass over a contiguous group of 14 (complex64) or 13 (complex128) qubits:
// the z phase between the group's transform and its way back.
//
// Such a group lets a 24-qubit state take two groups, two passes a step, but
// its tile is 128 KiB: the general pass kernel keeps it in LDS for its layout
// changes, one workgroup per CU, whose loads, six layout changes and stores
// follow one another (108 us on the 128 MiB complex64 state of a 3x4 torus,
// 2.5 TB/s).  Here the lane bits are transformed in the wave, and only the
// three wave bits pass through LDS, once each way and one component at a
// time (64 KiB), so two workgroups share a CU: 65 us, 4.1 TB/s (complex128:
// step of a 13 + 11 qubit plan 373 -> 301 us).  What is left is the order of
// load, transform and store within a workgroup; a copy in place of that size
// runs at 5.9 TB/s.  In complex64 the layers run in the general kernel's order
// (9-13, 4-8, 0-3 and back from the lowest window) and the norm's FP32 sums
// take its groups, so the bits are the same; in complex128 the windows differ
// and the two kernels agree to rounding.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "z2h_internal.h"
#include "z2h_kernels.h"
#include "z2h_sched.h"
#include "z2h_tile.h"
#include "z2h_wave.h"

namespace z2h {

namespace {

// Sum of |v|^2 over the block, after the forward layers.  FP32 over the five
// lowest index bits (pairwise from the highest, as the general pass sums a
// thread's 32 elements), FP64 over the others.
template <int RB, int WB, typename Real>
__device__ __forceinline__ double wave_norm(const Cx<Real> (&v)[1 << RB], double *red) {
    double s = 0.0;
#pragma unroll
    for (int k = 0; k < (1 << RB); k += 2) {
        Real a = abs2<true>(v[k]) + abs2<true>(v[k + 1]);
        a += lane_across<3>(a);
        a += lane_across<2>(a);
        a += lane_across<1>(a);
        a += lane_across<0>(a);
        s += (double)a;
    }
    double y = s;
    lane_swap<4>(s, y);
    s += y;
    y = s;
    lane_swap<5>(s, y);
    s += y;
    __syncthreads();
    if ((threadIdx.x & 63u) == 0) red[threadIdx.x >> 6] = s;
    __syncthreads();
    s = 0.0;
    for (int j = 0; j < (1 << WB); ++j) s += red[j];
    return s;
}

template <typename Real, int RB, int WB>
__global__ void __launch_bounds__(64 << WB) __attribute__((amdgpu_waves_per_eu(4))) wide_kernel(LevelArgs a) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    constexpr int m = RB + 6 + WB;
    const uint32_t t = threadIdx.x, lane = t & 63u, wave = t >> 6, lam = wave_lane(lane);
    const uint64_t bid = a.xcd ? xcd_major(blockIdx.x, gridDim.x) : blockIdx.x;
    const int jb = (int)(bid >> a.geom.tiles_log2);
    const uint64_t tile = bid & ((1ull << a.geom.tiles_log2) - 1);
    const int n = a.lat.n, nst = a.lat.nst;

    // (a uniform job stride: the loads go out before the record is read)
    Cx<Real> *st = reinterpret_cast<Cx<Real> *>(a.states) + a.jbase + (uint64_t)jb * a.jstride;
    const JobDev J = job_record(a.jobs, a.jidx ? job_index(a.jidx, jb) : jb, a.job_inline);
    const LevelOp op = level_op(a.level - J.lev0, a.K, J.steps, J.k_begin, J.order);
    if (op.kind != kPhaseB || op.group != a.group) return;  // uniform
    if (a.jmode != 0) st = reinterpret_cast<Cx<Real> *>(a.states) + J.offset;
    const uint32_t base = (uint32_t)(tile << m) | (wave << 6) | lam;
    Cx<Real> v[1 << RB];
#pragma unroll
    for (int q = 0; q < (1 << RB); ++q) v[q] = st[base + ((uint32_t)q << (6 + WB))];

    // exchange region (one component of the tile; the table's factors before
    // it is used), phase table, reduction
    Cx<Real> *lds = reinterpret_cast<Cx<Real> *>(smem);
    Cx<Real> *tab = reinterpret_cast<Cx<Real> *>(smem + ((size_t)sizeof(Real) << m));
    double *red = align16<double>(tab + (nst + 1) * (n + 1));
    double alpha, beta;
    phase_angles(J, op, alpha, beta);
    build_table<Real>(tab, table_scratch(smem), nst, n, alpha, beta, 1.0);
    LayCtx<RB> L;
    const uint32_t i0 = (uint32_t)(tile << m) | wave_index<RB, WB>(wave, lam, 0u);
    L.s0z = syndrome_direct(a.lat.zmask, i0);
    L.w0 = popc(i0);
#pragma unroll
    for (int r = 0; r < RB; ++r) L.lz[r] = a.lat.zsyn[wave_reg_bit<RB, WB>(r)];

    fwd_wave<RB, WB, true>(v, lds, wave, lane, lam);
    if (op.norm && (J.renorm || J.norm_trace)) {
        const double s = wave_norm<RB, WB>(v, red);
        if (t == 0 && J.norm_part) gst(J.norm_part, (int64_t)tile, s);
    }
    apply_phase<Real, RB>(v, L, 0, n, tab);
    bwd_wave<RB, WB, true>(v, lds, wave, lane, lam);

    uint32_t b = base;
    asm volatile("" : "+v"(b));
#pragma unroll
    for (int q = 0; q < (1 << RB); ++q) st[b + ((uint32_t)q << (6 + WB))] = v[q];
}

size_t wide_lds(const LatticeDev &lat, size_t real, int m) {
    return (real << m) + (((size_t)(lat.nst + 1) * (lat.n + 1) * 2 * real + 31) & ~(size_t)15) + 16 * sizeof(double);
}

template <typename Real, int RB, int WB>
hipError_t do_wide(const LevelArgs &a, unsigned nblocks, hipStream_t s) {
    const size_t lds = wide_lds(a.lat, sizeof(Real), RB + 6 + WB);
    hipError_t e = set_lds(reinterpret_cast<const void *>(&wide_kernel<Real, RB, WB>), lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((wide_kernel<Real, RB, WB>), dim3(nblocks), dim3(64 << WB), lds, s, a);
    return hipGetLastError();
}

}  // namespace

// Group 0 of 14 (complex64) or 13 (complex128) qubits, one tile per value of
// the others.
bool wide_level_ok(bool c128, const GroupGeom &g) {
    const int m = c128 ? 13 : 14;
    return !g.full && !g.hi && g.c == 0 && g.b0 == 0 && g.x0 == 0 && g.x1 == m && g.m == m && g.R == (c128 ? 4 : 5);
}

hipError_t prepare_wide() {
    hipError_t e = set_lds(reinterpret_cast<const void *>(&wide_kernel<float, 5, 3>), kMaxLdsBytes);
    if (e == hipSuccess) e = set_lds(reinterpret_cast<const void *>(&wide_kernel<double, 4, 3>), kMaxLdsBytes);
    return e;
}

hipError_t launch_wide(bool c128, const LevelArgs &a, unsigned nblocks, hipStream_t s) {
    if (!wide_level_ok(c128, a.geom)) return hipErrorInvalidValue;
    return c128 ? do_wide<double, 4, 3>(a, nblocks, s) : do_wide<float, 5, 3>(a, nblocks, s);
}

}  // namespace z2h
