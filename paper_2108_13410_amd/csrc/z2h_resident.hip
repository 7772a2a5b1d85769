// Whole ramps of small lattices (8 and 12 qubits) inside one workgroup: the
// state stays in registers from the first step to the last.
//
// The lowest six qubits are lane bits, the highest RB qubits register bits,
// and at 12 qubits the two between them wave bits.  Register and lane bits
// are transformed in the wave (z2h_wave.h); the wave bits come into the
// registers through LDS, one exchange each way.  The layers run in the order
// of the pass kernels' register windows (8-11, 4-7, 0-3 and back from the
// lowest window; 6-7, 4-5, 2-3, 0-1 at 8 qubits), so that rounding does not
// depend on how a layer is done.  The indices of an element's phase (odd stabilizers, weight) do
// not change over the ramp, so every thread keeps its table offsets.
//
// What bounds it is the serial chain of one step, not bytes or operations
// (one workgroup per state): so the tables come off that chain.  Their sines
// and cosines are computed for several phases at once, a wave for as many
// phases as its lanes hold factors, and at 8 qubits (one wave of amplitudes)
// by three further waves while the first one steps.
// Measured per step of one state (complex128 / complex64; before, with every
// layout change through LDS and the tables on the chain: 2.51 / 2.31 us at 8
// qubits, 8.1 / 4.9 us at 12): 0.91 / 0.74 us and 4.9 / 3.7 us, with
// renormalization 0.17 and 0.3 us more.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "z2h_internal.h"
#include "z2h_kernels.h"
#include "z2h_sched.h"
#include "z2h_tile.h"
#include "z2h_wave.h"

namespace z2h {

namespace {

// Shape of a state of RB + 6 + WB qubits: RB register bits, WB wave bits,
// PW waves that only build tables (0: the stepping waves build them between
// two chunks of phases), tables for at most CH phases at once.
template <int RB_, int WB_, int PW_, int CH>
struct Shape {
    static constexpr int RB = RB_, WB = WB_, PW = PW_;
    static constexpr int n = RB + 6 + WB, nst = n / 2, W = n + 1;
    static constexpr int entries = (nst + 1) * W, nfac = nst + 1 + W;
    static constexpr int step_waves = 1 << WB, waves = step_waves + PW;
    static constexpr int per_wave = 64 / nfac;                            // phases a wave builds at once
    static constexpr int chunk = CH;                                      // phases per chunk
    static_assert(CH <= per_wave * (PW ? PW : step_waves) && (!PW || CH == per_wave * PW), "who builds a chunk");
    static constexpr int threads = 64 * waves;
    static constexpr int bufs = PW ? 2 : 1;
};
typedef Shape<2, 0, 3, 12> Shape8;
typedef Shape<4, 2, 0, 12> Shape12;
typedef Shape<4, 2, 0, 11> Shape12Two;  // two workgroups per CU

// EX: exchange regions (with one, a barrier more each way).
template <typename S, typename Real, int EX>
struct Lds {
    double2 tab[S::bufs][S::chunk][S::entries];
    double red[S::step_waves];
    union {  // (stepping waves build tables between two steps, barriers on either side)
        double2 fac[S::waves][64];
        Cx<Real> ex[EX][S::WB ? (64 << (S::RB + S::WB)) : 1];
    };
};
// Launches of more states than the GPU has CUs run two workgroups per CU: the
// steps are chains of latencies, and a second chain fits between.  12 qubits,
// complex64: 231 registers a thread, and 80 KiB of LDS with 11 tables.
// Complex128: one exchange region (80 KiB), and 256 registers of the 346 that
// a workgroup alone takes (75 spilled, nearly all used between two steps
// only).  4096 ramps of 100 steps, one workgroup per CU against two: complex64
// 6.93 and 4.36 ms, complex128 8.38 and 6.87; 320 ramps 0.90 and 0.62, 1.07
// and 0.94; 256 ramps 0.49 and 0.50, 0.58 and 0.69.
constexpr unsigned kCUs = 256;
static_assert(2 * sizeof(Lds<Shape12Two, float, 2>) <= (size_t)kMaxLdsBytes &&
                  2 * sizeof(Lds<Shape12Two, double, 1>) <= (size_t)kMaxLdsBytes, "two workgroups per CU");

// Tables of phases p0 .. p0 + per_wave - 1, those below nph, of the ramp
// (phase p is level lev0 + p), by one wave, in FP64: T[k][w] = exp(i (alpha
// (nst - 2k) + beta (n - 2w))), times 2^-n in the Hadamard basis.  The
// factors pass between the wave's own lanes through LDS.
template <typename S>
__device__ __forceinline__ void build_phases(const JobDev &J, int lev0, int nph, int p0, double2 (*tab)[S::entries],
                                             double2 *fac, uint32_t lane) {
#pragma clang fp contract(off)
    const int own = (int)lane / S::nfac, j = (int)lane - own * S::nfac;
    if (own < S::per_wave && p0 + own < nph) {
        const LevelOp op = level_op(lev0 + p0 + own, 2, J.steps, J.k_begin, J.order);
        double alpha, beta;
        phase_angles(J, op, alpha, beta);
        const double ang = j <= S::nst ? alpha * (double)(S::nst - 2 * j) : beta * (double)(S::n - 2 * (j - S::nst - 1));
        double s, c;
        sincos(ang, &s, &c);
        fac[lane] = make_double2(c, s);
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    for (int i = (int)lane; i < S::per_wave * S::entries; i += 64) {
        const int q = i / S::entries, e = i - q * S::entries;
        if (p0 + q >= nph) break;
        const int k = e / S::W, w = e - k * S::W;
        const double2 a = fac[q * S::nfac + k], b = fac[q * S::nfac + S::nst + 1 + w];
        // levels alternate between the bases, odd ones in the Hadamard basis
        const double scale = ((lev0 + p0 + q) & 1) ? 1.0 / (double)(1 << S::n) : 1.0;
        tab[q][e] = make_double2((a.x * b.x - a.y * b.y) * scale, (a.x * b.y + a.y * b.x) * scale);
    }
    // (the next call's factors must not overtake these reads)
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Table offset of every register element's index i in one basis.
template <typename S>
__device__ __forceinline__ uint32_t table_index(const uint32_t *masks, uint32_t i) {
    uint32_t k = 0;
#pragma unroll
    for (int s = 0; s < S::nst; ++s) k += (uint32_t)(popc(i & masks[s]) & 1);
    return k * (uint32_t)S::W + (uint32_t)popc(i);
}

template <typename Real, int N>
__device__ __forceinline__ void phase(Cx<Real> (&v)[N], const uint32_t (&at)[N], const double2 *tab, double f) {
#pragma clang fp contract(off)
    Cx<Real> w[N];
#pragma unroll
    for (int q = 0; q < N; ++q) {
        const double2 e = tab[at[q]];
        w[q] = Cx<Real>{(Real)(e.x * f), (Real)(e.y * f)};
    }
    // (the multiply-adds spelled out: every phase rounds alike)
#pragma unroll
    for (int q = 0; q < N; ++q) {
        const Cx<Real> a = v[q];
        v[q].x = madd(a.x, w[q].x, -(a.y * w[q].y));
        v[q].y = madd(a.y, w[q].x, a.x * w[q].y);
    }
}

// Sum of |v|^2 over a thread's elements, pairwise in the storage precision.
// The first IM elements take the form abs2<true>: three in the x-z-x order
// at 12 qubits, none elsewhere, which are the sums (to the last bit) that
// renormalized complex64 ramps have been scaled by.
template <int IM, typename Real, int N>
__device__ __forceinline__ double reg_norm(const Cx<Real> (&v)[N]) {
    Real a[N];
#pragma unroll
    for (int q = 0; q < N; ++q) a[q] = q < IM ? abs2<true>(v[q]) : abs2<false>(v[q]);
#pragma unroll
    for (int h = N >> 1; h > 0; h >>= 1) {
#pragma unroll
        for (int q = 0; q < h; ++q) a[q] += a[q + h];
    }
    return (double)a[0];
}

template <typename S, typename Real, int EX>
__global__ void __launch_bounds__(S::threads) __attribute__((amdgpu_waves_per_eu(S::WB && EX == 1 ? 2 : 1)))
resident_kernel(ResidentArgs a) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    Lds<S, Real, EX> &L = *reinterpret_cast<Lds<S, Real, EX> *>(smem);
    const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6, lam = wave_lane(lane);
    const JobDev J = job_record(a.jobs, (int)blockIdx.x, a.job_inline);
    if (J.steps <= 0) return;  // uniform
    constexpr int N = 1 << S::RB;
    // phase p of the ramp is level lev0 + p: x z x .. x, or z x z .. z
    const int lev0 = J.order == 0 ? 1 : 0, nph = 2 * J.steps + 1;
    const bool steps = S::PW == 0 || wave < (uint32_t)S::step_waves;  // this wave holds amplitudes

    Cx<Real> v[N];
    uint32_t atz[N], atx[N];
    Cx<Real> *st = reinterpret_cast<Cx<Real> *>(a.states) + J.offset;
    const uint32_t base = (wave << 6) | lam;
    if (steps) {
#pragma unroll
        for (int q = 0; q < N; ++q) {
            const uint32_t i = base | ((uint32_t)q << (6 + S::WB));
            v[q] = st[i];
            atz[q] = table_index<S>(a.lat.zmask, i);
            atx[q] = table_index<S>(a.lat.xmask, wave_index<S::RB, S::WB>(wave, lam, (uint32_t)q));
        }
    }
    const bool use_norms = J.renorm || J.norm_trace;
    double norm = 1.0;      // of the last z phase
    bool have_norm = false;

    auto run = [&](int p, const double2 *tab) {
        const int lev = lev0 + p;
        if ((lev & 1) == 0) {  // computational basis
            const bool meas = use_norms && (J.order == 0 || p < nph - 1);
            if (meas) {
                const double s = wave_sum_lanes(S::WB && J.order == 0 ? reg_norm<3>(v) : reg_norm<0>(v));
                if constexpr (S::WB == 0) norm = s;
                else if (lane == 0) L.red[wave] = s;  // read after the next exchange's barrier
                have_norm = true;
            }
            phase<Real, N>(v, atz, tab, 1.0);
            return;
        }
        if constexpr (S::WB && EX == 1) __syncthreads();
        fwd_wave<S::RB, S::WB, false>(v, L.ex[0], wave, lane, lam);
        double f = 1.0;
        if (have_norm) {
            if constexpr (S::WB != 0) {
                norm = 0.0;
                for (int j = 0; j < S::step_waves; ++j) norm += L.red[j];
            }
            if (threadIdx.x == 0 && J.norm_trace)
                gst(J.norm_trace, J.order == 0 ? p / 2 - 1 : p / 2, norm);
            if (J.renorm) f = 1.0 / sqrt(norm);
        }
        phase<Real, N>(v, atx, tab, f);
        if constexpr (S::WB && EX == 1) __syncthreads();
        bwd_wave<S::RB, S::WB, false>(v, L.ex[EX - 1], wave, lane, lam);
    };

    if constexpr (S::PW != 0) {
        const int pw = (int)wave - S::step_waves;
        if (pw >= 0) build_phases<S>(J, lev0, nph, pw * S::per_wave, &L.tab[0][pw * S::per_wave], L.fac[wave], lane);
        __syncthreads();
        for (int c = 0; c * S::chunk < nph; ++c) {
            if (steps) {
                const int hi = nph - c * S::chunk < S::chunk ? nph - c * S::chunk : S::chunk;
                for (int p = 0; p < hi; ++p) run(c * S::chunk + p, L.tab[c & 1][p]);
            } else {
                build_phases<S>(J, lev0, nph, (c + 1) * S::chunk + pw * S::per_wave,
                                &L.tab[(c + 1) & 1][pw * S::per_wave], L.fac[wave], lane);
            }
            __syncthreads();
        }
    } else {
        for (int c = 0; c < nph; c += S::chunk) {
            __syncthreads();  // the last chunk's tables are no longer read
            const int hi = nph - c < S::chunk ? nph - c : S::chunk;
            build_phases<S>(J, lev0, c + hi, c + (int)wave * S::per_wave, &L.tab[0][wave * S::per_wave], L.fac[wave], lane);
            __syncthreads();
            for (int p = 0; p < hi; ++p) run(c + p, L.tab[0][p]);
        }
    }
    if (steps) {
#pragma unroll
        for (int q = 0; q < N; ++q) st[base | ((uint32_t)q << (6 + S::WB))] = v[q];
    }
}

template <typename S, typename Real, int EX>
hipError_t do_resident(const ResidentArgs &a, unsigned njobs, hipStream_t s) {
    constexpr size_t lds = sizeof(Lds<S, Real, EX>);
    static_assert(lds <= (size_t)kMaxLdsBytes, "LDS of one workgroup");
    hipError_t e = set_lds(reinterpret_cast<const void *>(&resident_kernel<S, Real, EX>), lds);
    if (e != hipSuccess || !njobs) return e;
    hipLaunchKernelGGL((resident_kernel<S, Real, EX>), dim3(njobs), dim3(S::threads), lds, s, a);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_resident(bool c128, const ResidentArgs &a, unsigned njobs, hipStream_t s) {
    if (a.lat.n == Shape8::n) return c128 ? do_resident<Shape8, double, 1>(a, njobs, s) : do_resident<Shape8, float, 1>(a, njobs, s);
    if (a.lat.n != Shape12::n) return hipErrorInvalidValue;
    if (njobs > kCUs) return c128 ? do_resident<Shape12Two, double, 1>(a, njobs, s) : do_resident<Shape12Two, float, 2>(a, njobs, s);
    return c128 ? do_resident<Shape12, double, 2>(a, njobs, s) : do_resident<Shape12, float, 2>(a, njobs, s);
}

// The dynamic-LDS limits only (no launch).
hipError_t prepare_resident() {
    ResidentArgs a{};
    hipError_t e = do_resident<Shape8, float, 1>(a, 0, nullptr);
    if (e == hipSuccess) e = do_resident<Shape8, double, 1>(a, 0, nullptr);
    if (e == hipSuccess) e = do_resident<Shape12, float, 2>(a, 0, nullptr);
    if (e == hipSuccess) e = do_resident<Shape12, double, 2>(a, 0, nullptr);
    if (e == hipSuccess) e = do_resident<Shape12Two, float, 2>(a, 0, nullptr);
    if (e == hipSuccess) e = do_resident<Shape12Two, double, 1>(a, 0, nullptr);
    return e;
}

}  // namespace z2h
