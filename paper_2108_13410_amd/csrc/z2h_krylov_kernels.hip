// Device kernels of the exact solvers of libz2h: the Hamiltonian of the
// mapped model (Sec. II, Eq. effi) applied to a state, and the vector
// operations of the Lanczos recurrence that the ground-energy and Krylov
// time-evolution entry points build on (the exact references of Sec. VII).
//
// H = D_Z + 2^-n W D_X W, with W the unnormalised Walsh-Hadamard transform
// over all links, D_Z(i) = -JB (nst - 2 k_p(i)) - hz (n - 2 w(i)) the
// plaquette and z-field terms in the computational basis and D_X the star and
// x-field terms in the Hadamard basis (same form with k_v and hx).  The
// transform reuses the tile passes of the Trotter step: one pass per group
// up to the top group, which multiplies by D_X between its forward and
// backward transform, and one pass per group back down; the last pass adds
// D_Z x.  Nothing is exponentiated, so the diagonal is computed per element
// from the syndrome and the Hamming weight.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <mutex>
#include <set>

#include "z2h_internal.h"
#include "z2h_kernels.h"
#include "z2h_solvers.h"
#include "z2h_tile.h"
#include "z2h_wave.h"

namespace z2h {

// Value of one basis' diagonal at syndrome s and weight w.
__device__ __forceinline__ double diag_value(int nst, int n, uint32_t s, int w, double J, double h) {
    return -(J * (double)(nst - 2 * popc(s)) + h * (double)(n - 2 * w));
}

// v *= scale * D_X for the register elements of layout L (Hadamard basis);
// accx (if not null) accumulates scale * sum D_X |v|^2 of the values before
// (a pointer: the accumulator then lives in a scratch slot rather than in
// one of the registers the two prefetched tiles need).  At most C elements'
// diagonals are live at a time.
template <typename Real, int R, int C = 1 << R>
__device__ __forceinline__ void mul_diag_x(Cx<Real> (&v)[1 << R], const LayCtx<R> &L, const LatticeDev &lat,
                                           double J, double h, double scale, double *accx) {
    uint32_t s = L.s0x;
#pragma unroll
    for (int idx = 0; idx < (1 << R); ++idx) {
        const int q = idx ^ (idx >> 1);
        if (idx) s ^= L.lx[__builtin_ctz(idx)];
        const double dd = scale * diag_value(lat.nst, lat.n, s, L.w0 + __builtin_popcount(q), J, h);
        if (accx) *accx += dd * ((double)v[q].x * (double)v[q].x + (double)v[q].y * (double)v[q].y);
        const Real d = (Real)dd;
        v[q].x *= d;
        v[q].y *= d;
        if constexpr (C < (1 << R))
            if (idx % C == C - 1) __builtin_amdgcn_sched_barrier(0);
    }
}

// sum D_Z |v|^2 over the register elements of layout L (computational basis).
template <typename Real, int R>
__device__ __forceinline__ double diag_norm_z(const Cx<Real> (&v)[1 << R], const LayCtx<R> &L,
                                              const LatticeDev &lat, double J, double h) {
    uint32_t s = L.s0z;
    double acc = 0.0;
#pragma unroll
    for (int idx = 0; idx < (1 << R); ++idx) {
        const int q = idx ^ (idx >> 1);
        if (idx) s ^= L.lz[__builtin_ctz(idx)];
        acc += diag_value(lat.nst, lat.n, s, L.w0 + __builtin_popcount(q), J, h) *
               ((double)v[q].x * (double)v[q].x + (double)v[q].y * (double)v[q].y);
    }
    return acc;
}

// Elements of x at the register positions of layout L, eight Gray-code steps
// at a time (each chunk covers eight register elements), so that at most
// eight extra elements of each operand are live beside the tile.
template <int R>
struct Chunk {
    static constexpr int C = (1 << R) < 8 ? (1 << R) : 8;
};

// v += D_Z x for the register elements of layout L (computational basis),
// accumulating Re(conj(x) v) of the result.
template <typename Real, int R, bool SP>
__device__ __forceinline__ void add_diag_z(Cx<Real> (&v)[1 << R], const Cx<Real> *x, const LayCtx<R> &L,
                                           const LatticeDev &lat, double J, double h, double &acc) {
    constexpr int C = Chunk<R>::C;
    uint32_t s = L.s0z;
    const Cx<Real> *b = x + L.i0;
#pragma unroll
    for (int c0 = 0; c0 < (1 << R); c0 += C) {
        Cx<Real> xv[C];
#pragma unroll
        for (int i = 0; i < C; ++i) {
            const int q = (c0 + i) ^ ((c0 + i) >> 1);
            xv[i] = b[reg_off<R, SP>(L, q)];
        }
#pragma unroll
        for (int i = 0; i < C; ++i) {
            const int idx = c0 + i, q = idx ^ (idx >> 1);
            if (idx) s ^= L.lz[__builtin_ctz(idx)];
            const Real d = (Real)diag_value(lat.nst, lat.n, s, L.w0 + __builtin_popcount(q), J, h);
            v[q].x += d * xv[i].x;
            v[q].y += d * xv[i].y;
            acc += (double)xv[i].x * (double)v[q].x + (double)xv[i].y * (double)v[q].y;
        }
        __builtin_amdgcn_sched_barrier(0);
    }
}

// Lanczos form of the last pass: with v = (2^-n W D_X W u) at the register
// positions of layout L, write w = sig (v + D_Z u - alpha u) - cp p and
// accumulate |w|^2.
template <typename Real, int R, bool SP>
__device__ __forceinline__ void lanczos_out(const Cx<Real> (&v)[1 << R], const Cx<Real> *u, const Cx<Real> *p,
                                            Cx<Real> *w, const LayCtx<R> &L, const LatticeDev &lat, double J,
                                            double h, double sig, double alpha, double cp, bool use_prev,
                                            double &acc) {
    constexpr int C = Chunk<R>::C;
    uint32_t s = L.s0z;
    const Cx<Real> *bu = u + L.i0;
    const Cx<Real> *bp = p + L.i0;
    Cx<Real> *bw = w + L.i0;
    const Real rs = (Real)sig, rc = (Real)cp;
#pragma unroll
    for (int c0 = 0; c0 < (1 << R); c0 += C) {
        Cx<Real> uv[C], pv[C];
#pragma unroll
        for (int i = 0; i < C; ++i) {
            const int q = (c0 + i) ^ ((c0 + i) >> 1);
            uv[i] = bu[reg_off<R, SP>(L, q)];
            pv[i] = use_prev ? bp[reg_off<R, SP>(L, q)] : Cx<Real>{(Real)0, (Real)0};
        }
#pragma unroll
        for (int i = 0; i < C; ++i) {
            const int idx = c0 + i, q = idx ^ (idx >> 1);
            if (idx) s ^= L.lz[__builtin_ctz(idx)];
            const Real d = (Real)(diag_value(lat.nst, lat.n, s, L.w0 + __builtin_popcount(q), J, h) - alpha);
            Cx<Real> r{rs * (v[q].x + d * uv[i].x) - rc * pv[i].x, rs * (v[q].y + d * uv[i].y) - rc * pv[i].y};
            bw[reg_off<R, SP>(L, q)] = r;
            acc += (double)r.x * (double)r.x + (double)r.y * (double)r.y;
        }
        __builtin_amdgcn_sched_barrier(0);
    }
}

// A value that every lane of the block holds alike, moved to scalar registers.
__device__ __forceinline__ double uniform(double x) {
    const uint64_t u = __builtin_bit_cast(uint64_t, x);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)u);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(u >> 32));
    return __builtin_bit_cast(double, (uint64_t)lo | ((uint64_t)hi << 32));
}

// Lanczos coefficients of this iteration: sigma_k, alpha_k and
// cp = beta_k sigma_{k-1}.  Every block sums the partials of the first and
// the top pass itself, and, where prev_w is given, beta_k and sigma_k from
// the last iteration's |w|^2 partials; block 0 then records them (a launch of
// one block between two iterations took 4 us, 10 us for 2048 partials).
__device__ __forceinline__ void lanczos_coefs(const HamArgs &a, double *red, double &sig, double &alpha, double &cp) {
    const int t = (int)threadIdx.x, nt = (int)blockDim.x;
    double sm = 0.0;
    for (int j = t; j < a.napart_z; j += nt) sm += a.apart_z[j];
    for (int j = t; j < a.napart_x; j += nt) sm += a.apart_x[j];
    double beta;
    if (a.prev_w) {
        double sw = 0.0;
        for (int j = t; j < a.nprev_w; j += nt) sw += a.prev_w[j];
        beta = uniform(sqrt(block_sum(sw, red)));
        sig = beta > 1e-300 ? 1.0 / beta : 0.0;
    } else {
        beta = a.coef[a.k].beta;
        sig = a.coef[a.k].sigma;
    }
    sig = uniform(sig);
    alpha = uniform(sig * sig * block_sum(sm, red));
    cp = a.use_prev ? beta * a.coef[a.k - 1].sigma : 0.0;
    if (a.record && blockIdx.x == 0 && t == 0) {
        a.coef[a.k].alpha = alpha;
        if (a.prev_w) {  // (else they are there, and other blocks read them)
            a.coef[a.k].beta = beta;
            a.coef[a.k].sigma = sig;
        }
    }
}

// Two complex128 tiles of 16 elements are the register limit: the plaquette
// masks are taken one at a time there.  All at once, held in scalar registers
// through the tile loop, they spilled 10 vector registers: a 4x4 product took
// 166.6 ms, a Lanczos iteration 181.5, now 157.8 and 170.4.  Other shapes have
// room for all masks, which is 1% to 2% faster.
template <typename Real, int R, bool PF>
constexpr bool two_tile_limit = PF && sizeof(Real) == 8 && R == 4;

// PF: the next tile's elements are loaded while the current one is
// transformed (two register tiles; used where they fit without spilling).
template <typename Real, int R, bool PF, bool SP>
__global__ void __launch_bounds__(512) ham_kernel(HamArgs a) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const GroupGeom &g = a.geom;
    const uint32_t t = threadIdx.x;
    const uint64_t tiles = 1ull << g.tiles_log2;
    Cx<Real> *lds = reinterpret_cast<Cx<Real> *>(smem);
    const uint32_t lds_elems = (1u << g.m) + (1u << (g.m - R));
    double *red = reinterpret_cast<double *>(lds + lds_elems);
    const Cx<Real> *src = reinterpret_cast<const Cx<Real> *>(a.src);
    Cx<Real> *dst = reinterpret_cast<Cx<Real> *>(a.dst);
    const Cx<Real> *x = reinterpret_cast<const Cx<Real> *>(a.x);
    const bool lz = a.lz && a.final_pass;
    double acc = 0.0, accz = 0.0, accx = 0.0;

    double sig = 0.0, alpha = 0.0, cp = 0.0;
    if (lz) lanczos_coefs(a, red, sig, alpha, cp);

    constexpr bool kLoop = two_tile_limit<Real, R, PF>;
    const bool syn0 = a.final_pass || a.part_z;
    // logical block: first tile of the grid-stride walk and partial slot
    const uint32_t lb = a.xcd ? xcd_major(blockIdx.x, gridDim.x) : blockIdx.x;
    uint64_t tile = lb;
    Cx<Real> vn[PF ? (1 << R) : 1];
    LayCtx<R> Ln;
    if constexpr (PF) {
        if (tile < tiles) {
            lay_ctx<R, SP, kLoop>(Ln, g, a.lat, tile, g.p[0], t, syn0, 0);
            load_tile<Real, R, false, SP>(vn, src, Ln);
        }
    }
    for (; tile < tiles; tile += gridDim.x) {
        Cx<Real> v[1 << R];
        LayCtx<R> L0;
        if constexpr (PF) {
            L0 = Ln;
#pragma unroll
            for (int q = 0; q < (1 << R); ++q) v[q] = vn[q];
            const uint64_t nt = tile + gridDim.x;
            if (nt < tiles) {
                lay_ctx<R, SP, kLoop>(Ln, g, a.lat, nt, g.p[0], t, syn0, 0);
                load_tile<Real, R, false, SP>(vn, src, Ln);
            }
        } else {
            lay_ctx<R, SP>(L0, g, a.lat, tile, g.p[0], t, syn0, 0);
            load_tile<Real, R, false, SP>(v, src, L0);
        }
        if (a.part_z) accz += diag_norm_z<Real, R>(v, L0, a.lat, a.JB, a.hz);
        int cur = 0;
        for (int j = 0; j < g.nlay; ++j) {
            if (j > 0) exchange<Real, R>(v, lds, g.p[j - 1], g.p[j], t);
            butterflies<Real, R>(v, g.blo[j], g.bhi[j]);
            cur = j;
        }
        if (a.top) {
            LayCtx<R> Lm;
            lay_ctx<R, SP>(Lm, g, a.lat, tile, g.p[cur], t, true, 1);
            mul_diag_x<Real, R>(v, Lm, a.lat, a.JA, a.hx, a.xscale, a.part_x ? &accx : nullptr);
            for (int j = g.nlay - 1; j >= 0; --j) {
                if (j != cur) {
                    exchange<Real, R>(v, lds, g.p[cur], g.p[j], t);
                    cur = j;
                }
                butterflies<Real, R>(v, g.blo[j], g.bhi[j]);
            }
        }
        if (cur != 0) exchange<Real, R>(v, lds, g.p[cur], g.p[0], t);
        if (lz) {
            lanczos_out<Real, R, SP>(v, x, reinterpret_cast<const Cx<Real> *>(a.p), reinterpret_cast<Cx<Real> *>(a.w),
                                 L0, a.lat, a.JB, a.hz, sig, alpha, cp, a.use_prev != 0, acc);
            continue;
        }
        if (a.final_pass) add_diag_z<Real, R, SP>(v, x, L0, a.lat, a.JB, a.hz, acc);
        store_tile<Real, R, false, SP>(v, dst, L0);
    }
    if (a.part) {
        const double s = block_sum(acc, red);
        if (t == 0) a.part[lb] = s;
    }
    if (a.part_w) {
        const double s = block_sum(acc, red);
        if (t == 0) a.part_w[lb] = s;
    }
    if (a.part_z) {
        const double s = block_sum(accz, red);
        if (t == 0) a.part_z[lb] = s;
    }
    if (a.part_x) {
        const double s = block_sum(accx, red);
        if (t == 0) a.part_x[lb] = s;
    }
}

// Passes of y = H x over a complex128 state of N qubits in two groups, the
// low and the high ones, three a product: ROLE 0 the low group forward, 1 the
// high group with the X-basis diagonal, 2 and 3 the low group's way back with
// the Lanczos update or with D_Z x added; 4 is 2 with the Ritz vector's sum of
// the two vectors it reads.  Six bits are transformed in the wave, WB wave
// bits through LDS once each way; the state between two passes stays in the
// order the transform leaves it in (the same addresses), with the signs that
// lane_layer defers.
//
// 24 qubits: 13 + 11, where the plan's narrower groups take five passes.  A
// tile of 2^13 elements is 128 KiB; in ham_kernel it fills the LDS (one
// workgroup per CU, four layout changes a pass, and three such passes take as
// long as five of 2^12).  Here one component at a time passes through half of
// that LDS, so two workgroups share a CU and walk four tiles each, the
// coefficients summed once from 512 partials.  Tiles of the high group hold
// 64-byte runs; neighbours meet in one XCD's L2.  At 256 MiB a pass takes
// 101 us (5.3 TB/s; a large copy 4.6, in place 5.9), 110 us (158 without the
// row mixing below), 212 us for the update's four streams and 318 us for six;
// a Lanczos iteration 649 -> 433 us, and 2 x 134 us less of separate
// accumulation per two vectors for 106 us more here.  Two elements of each
// operand at a time in the update: with four the registers spill (role 4:
// 406 us).
//
// 16 to 20 qubits: a pass is a chain of latencies (launch, tile, transform,
// store), with few waves per CU.  Tiles are small (2^9 of one wave, without
// any exchange, or 2^11 of four), and every operand is fetched at once before
// the transform.  The three passes at 18 qubits, 3 x 10.4 us in ham_kernel:
// 5.2 + 5.3 + 7.7 as 11 + 7 qubits, 5.0 + 8.1 + 6.9 as 9 + 9, 4.6 + 7.4 + 6.7
// as 10 + 8 with four registers, 5.3 + 8.3 + 9.8 as 10 + 8 with sixteen.
template <int N> struct HamShape {};
template <> struct HamShape<16> { static constexpr int RB = 3, LOW = 0, HIGH = 0; };
template <> struct HamShape<18> { static constexpr int RB = 3, LOW = 2, HIGH = 0; };
template <> struct HamShape<20> { static constexpr int RB = 3, LOW = 2, HIGH = 2; };
template <> struct HamShape<24> { static constexpr int RB = 4, LOW = 3, HIGH = 3; };

// Of the passes over one group: wave bits, tile qubits, threads per block,
// tiles per block (waves that share none of their tile), carried qubits.
template <int N, bool high>
struct HamTile {
    using S = HamShape<N>;
    static constexpr int RB = S::RB, WB = high ? S::HIGH : S::LOW, M = RB + 6 + WB, LOWQ = RB + 6 + S::LOW;
    static constexpr int C = high ? M - (N - LOWQ) : 0, T = WB ? 64 << WB : 128, per = WB ? 1 : 2;
    static constexpr bool wide = N == 24;
    static constexpr uint32_t tiles = 1u << (N - M);
    static constexpr uint32_t blocks = wide ? 512u : tiles / per;
    static constexpr size_t buf = WB ? (wide ? sizeof(double) : sizeof(Cx<double>)) << M : 0;  // exchange
};

template <int ROLE, int N>
__device__ __forceinline__ void ham_wave_body(const HamArgs &a) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    constexpr bool high = ROLE == 1, lanczos = ROLE == 2 || ROLE == 4;
    using G = HamTile<N, high>;
    constexpr int RB = G::RB, WB = G::WB, M = G::M, C = G::C, LOWQ = G::LOWQ;
    constexpr bool CX = G::wide;
    constexpr uint32_t CH = G::wide ? 2 : 1u << RB;  // operand elements at a time
    using V = Cx<double>;
    V *lds = reinterpret_cast<V *>(smem);
    double *red = reinterpret_cast<double *>(smem + G::buf);
    const uint32_t lane = threadIdx.x & 63u, wave = WB ? threadIdx.x >> 6 : 0u, lam = wave_lane(lane);
    const V *src = reinterpret_cast<const V *>(a.src), *x = reinterpret_cast<const V *>(a.x);
    V *dst = reinterpret_cast<V *>(a.dst);
    const uint32_t lb = G::wide ? xcd_major(blockIdx.x, gridDim.x) : blockIdx.x;
    double acc = 0.0, sig = 0.0, alpha = 0.0, cp = 0.0;
    if constexpr (lanczos && G::wide) lanczos_coefs(a, red, sig, alpha, cp);
    // Tile index of the thread's element q: nat(q) | nat_t as the transform
    // starts, fin(q) | fin_t as it ends; at() maps it to the state's (the
    // high group's tile holds 2^C neighbours of each of its elements).  The q
    // part of an address is uniform, the thread's byte offset fits 32 bits.
    const uint32_t nat_t = (wave << 6) | lam, fin_t = wave_index<RB, WB>(wave, lam, 0u);
    auto at = [](uint32_t i) -> uint32_t { return high ? (i & ((1u << C) - 1u)) | ((i >> C) << LOWQ) : i; };
    auto nat = [&](uint32_t q) { return at(q << (6 + WB)); };
    auto fin = [&](uint32_t q) { return at(wave_index<RB, WB>(0u, 0u, q)); };
    constexpr uint32_t low = (1u << C) - 1u, row = (1u << LOWQ) - 1u;
    constexpr uint32_t nat_q = row & ~((1u << (6 + WB - C + 3)) - 1u);
    constexpr uint32_t fin_q = wave_index<RB, WB>(0u, 0u, (1u << RB) - 1u);
    uint32_t tile = lb;
    if constexpr (WB == 0) tile = lb * G::per + (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    for (; tile < G::tiles; tile += gridDim.x * G::per) {
        const uint32_t t0 = high ? tile << C : tile << M;
        auto elem = [&](const V *b, uint32_t u, uint32_t off) -> const V & {
            return *reinterpret_cast<const V *>(reinterpret_cast<const char *>(b + u) + off);
        };
        // 24 qubits: between the passes the element of the high index h and
        // the low index l sits at l ^ (h << 3): the high group's rows,
        // 128 KiB apart, then start in different memory channels.
        auto mix = [](uint32_t h) -> uint32_t { return G::wide ? (h << 3) & row : 0u; };
        auto y_q = [&](uint32_t q) -> uint32_t {
            return high ? nat(q) | ((t0 ^ mix((q << (6 + WB)) >> C)) & nat_q) : t0 | (fin(q) ^ (mix(tile) & fin_q));
        };
        const uint32_t y_t =
            high ? at(nat_t & ~low) | (((t0 ^ mix(nat_t >> C)) & (row & ~nat_q)) | (nat_t & low)) : fin_t ^ (mix(tile) & ~fin_q);
        const uint32_t nat_b = nat_t * (uint32_t)sizeof(V), y_b = y_t * (uint32_t)sizeof(V);
        V v[1 << RB];
#pragma unroll
        for (uint32_t q = 0; q < (1u << RB); ++q) v[q] = ROLE == 0 ? elem(src, t0 | nat(q), nat_b) : elem(src, y_q(q), y_b);

        // operands of the update (g: read as x and taken zero times at first)
        const V *p = reinterpret_cast<const V *>(a.use_prev ? a.p : a.x);  // (cp = 0 without one)
        V *w = lanczos ? reinterpret_cast<V *>(a.w) : dst, *gout = reinterpret_cast<V *>(a.g);
        const V *g = a.g_first ? x : gout;
        const double gf = a.g_first ? 0.0 : 1.0;
        V xv[CH], pv[CH], gv[CH];
        auto fetch = [&](uint32_t c0, uint32_t off) {
#pragma unroll
            for (uint32_t i = 0; i < CH; ++i) {
                const uint32_t q = (c0 + i) ^ ((c0 + i) >> 1);
                if constexpr (ROLE >= 2) xv[i] = elem(x, t0 | nat(q), off);
                if constexpr (lanczos) pv[i] = elem(p, t0 | nat(q), off);
                if constexpr (ROLE == 4 && !G::wide) gv[i] = elem(g, t0 | nat(q), off);
            }
        };
        if constexpr (!G::wide) fetch(0, nat_b);
        if constexpr (lanczos && !G::wide) lanczos_coefs(a, red, sig, alpha, cp);
        const double g0 = ROLE == 4 ? a.gs[0] * a.coef[a.k - 1].sigma : 0.0, g1 = ROLE == 4 ? a.gs[1] * sig : 0.0;

        LayCtx<RB> L;
        const uint32_t i0 = t0 | at(high ? fin_t : nat_t);
        L.w0 = popc(i0);
        if constexpr (high) {
            L.s0x = syndrome_direct(a.lat.xmask, i0);
#pragma unroll
            for (int r = 0; r < RB; ++r) L.lx[r] = a.lat.xsyn[wave_reg_bit<RB, WB>(r) - C + LOWQ];
            fwd_wave<RB, WB, CX, C>(v, lds, wave, lane, lam);
            mul_diag_x<double, RB, 4>(v, L, a.lat, a.JA, a.hx, a.xscale, &acc);
            if constexpr (WB && !CX) __syncthreads();
            bwd_wave<RB, WB, CX, C>(v, lds, wave, lane, lam);
        } else {
            L.s0z = syndrome_direct(a.lat.zmask, i0);
#pragma unroll
            for (int r = 0; r < RB; ++r) L.lz[r] = a.lat.zsyn[6 + WB + r];
            if constexpr (ROLE == 0) {
                if (a.part_z) acc += diag_norm_z<double, RB>(v, L, a.lat, a.JB, a.hz);
                fwd_wave<RB, WB, CX>(v, lds, wave, lane, lam);
            } else {
                bwd_wave<RB, WB, CX>(v, lds, wave, lane, lam);
            }
        }
        uint32_t ob = ROLE < 2 ? y_b : nat_b;
        asm volatile("" : "+v"(ob));  // (addresses are formed again, not kept)
        if constexpr (ROLE < 2) {
#pragma unroll
            for (uint32_t q = 0; q < (1u << RB); ++q) const_cast<V &>(elem(dst, y_q(q), ob)) = v[q];
        } else {
            // + D_Z x, CH elements of each operand at a time
            uint32_t s = L.s0z;
#pragma unroll
            for (uint32_t c0 = 0; c0 < (1u << RB); c0 += CH) {
                if constexpr (G::wide) fetch(c0, ob);
#pragma unroll
                for (uint32_t i = 0; i < CH; ++i) {
                    const uint32_t idx = c0 + i, q = idx ^ (idx >> 1);
                    if (idx) s ^= L.lz[__builtin_ctz(idx)];
                    const double d = diag_value(a.lat.nst, a.lat.n, s, L.w0 + popc(q), a.JB, a.hz);
                    V r{v[q].x + (d - alpha) * xv[i].x, v[q].y + (d - alpha) * xv[i].y};
                    if constexpr (lanczos) {
                        r = V{sig * r.x - cp * pv[i].x, sig * r.y - cp * pv[i].y};
                        acc += r.x * r.x + r.y * r.y;
                    } else {
                        acc += xv[i].x * r.x + xv[i].y * r.y;
                    }
                    const_cast<V &>(elem(w, t0 | nat(q), ob)) = r;
                }
                if constexpr (ROLE == 4) {
                    if constexpr (G::wide) {
#pragma unroll
                        for (uint32_t i = 0; i < CH; ++i) gv[i] = elem(g, t0 | nat((c0 + i) ^ ((c0 + i) >> 1)), ob);
                    }
#pragma unroll
                    for (uint32_t i = 0; i < CH; ++i) {
                        const V o{gf * gv[i].x + g0 * pv[i].x, gf * gv[i].y + g0 * pv[i].y};
                        const_cast<V &>(elem(gout, t0 | nat((c0 + i) ^ ((c0 + i) >> 1)), ob)) =
                            V{o.x + g1 * xv[i].x, o.y + g1 * xv[i].y};
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }
    double *part = ROLE == 0 ? a.part_z : ROLE == 1 ? a.part_x : lanczos ? a.part_w : a.part;
    if (part) {
        const double s = block_sum(acc, red);
        if (threadIdx.x == 0) part[lb] = s;
    }
}

template <int ROLE, int N>
__global__ void __launch_bounds__((HamTile<N, (ROLE == 1)>::T)) ham_wave_kernel(HamArgs a) {
    ham_wave_body<ROLE, N>(a);
}
// (two workgroups of 512 threads per CU)
template <int ROLE>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(4))) ham_wide_kernel(HamArgs a) {
    ham_wave_body<ROLE, 24>(a);
}

// Deterministic sum of n partials by one block (every thread gets it).
__device__ double sum_parts(const double *p, int n, double *red) {
    double s = 0.0;
    for (int j = (int)threadIdx.x; j < n; j += (int)blockDim.x) s += p[j];
    return block_sum(s, red);
}

template <typename Real>
__global__ void __launch_bounds__(256) vec_kernel(VecArgs a) {
    __shared__ double red[8];
    const Cx<Real> *y = reinterpret_cast<const Cx<Real> *>(a.y);
    const Cx<Real> *u = reinterpret_cast<const Cx<Real> *>(a.u);
    const Cx<Real> *p = reinterpret_cast<const Cx<Real> *>(a.p);
    Cx<Real> *w = reinterpret_cast<Cx<Real> *>(a.w);
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    double acc = 0.0;
    if (a.mode == 1) {
        for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < a.nelem; i += stride) {
            const Cx<Real> e = u[i];
            acc += (double)e.x * (double)e.x + (double)e.y * (double)e.y;
        }
    } else {
        const LanczosCoef ck = a.coef[a.k];
        const double sig = ck.sigma;
        const double alpha = sig * sig * sum_parts(a.apart, a.napart, red);
        const Real cy = (Real)sig, cu = (Real)(alpha * sig);
        const Real cp = a.use_prev ? (Real)(ck.beta * a.coef[a.k - 1].sigma) : (Real)0;
        for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < a.nelem; i += stride) {
            const Cx<Real> ey = y[i], eu = u[i];
            Cx<Real> r{cy * ey.x - cu * eu.x, cy * ey.y - cu * eu.y};
            if (a.use_prev) {
                const Cx<Real> ep = p[i];
                r.x -= cp * ep.x;
                r.y -= cp * ep.y;
            }
            w[i] = r;
            acc += (double)r.x * (double)r.x + (double)r.y * (double)r.y;
        }
    }
    const double s = block_sum(acc, red);
    if (threadIdx.x == 0) a.part[blockIdx.x] = s;
}

__global__ void __launch_bounds__(256) scalar_kernel(ScalarArgs a) {
    __shared__ double red[8];
    if (a.mode == 1) {
        const double nn = sum_parts(a.wpart, a.nwpart, red);
        if (threadIdx.x == 0) {
            const double b = sqrt(nn);
            a.coef[0] = LanczosCoef{0.0, b, b > 1e-300 ? 1.0 / b : 0.0, 0.0};
        }
        return;
    }
    const double sig = a.coef[a.k].sigma;
    const double alpha = sig * sig * (sum_parts(a.apart, a.napart, red) + sum_parts(a.apart2, a.napart2, red));
    const double nn = sum_parts(a.wpart, a.nwpart, red);
    if (threadIdx.x == 0) {
        a.coef[a.k].alpha = alpha;
        const double b = sqrt(nn);
        a.coef[a.k + 1] = LanczosCoef{0.0, b, b > 1e-300 ? 1.0 / b : 0.0, 0.0};
    }
}

template <typename Real>
__global__ void __launch_bounds__(256) combine_kernel(CombineArgs a) {
    Cx<Real> *psi = reinterpret_cast<Cx<Real> *>(a.psi);
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < a.nelem; i += stride) {
        double re = 0.0, im = 0.0;
        for (int j = 0; j < a.m; ++j) {
            const Cx<Real> e = reinterpret_cast<const Cx<Real> *>(a.u[j])[i];
            re += a.cre[j] * (double)e.x - a.cim[j] * (double)e.y;
            im += a.cre[j] * (double)e.y + a.cim[j] * (double)e.x;
        }
        psi[i] = Cx<Real>{(Real)re, (Real)im};
    }
}

template <typename Real>
__global__ void __launch_bounds__(256) acc_kernel(AccArgs a) {
    Cx<Real> *g = reinterpret_cast<Cx<Real> *>(a.g);
    const Cx<Real> *u = reinterpret_cast<const Cx<Real> *>(a.u);
    const Cx<Real> *u2 = reinterpret_cast<const Cx<Real> *>(a.u2);
    const double c = a.s * a.coef[a.k].sigma;
    const double c2 = u2 ? a.s2 * a.coef[a.k + 1].sigma : 0.0;
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < a.nelem; i += stride) {
        const Cx<Real> e = u[i];
        double re = c * (double)e.x, im = c * (double)e.y;
        if (!a.first) {
            const Cx<Real> o = g[i];
            re += (double)o.x;
            im += (double)o.y;
        }
        if (u2) {  // (rounded in between, as two launches would)
            const Cx<Real> f = u2[i];
            re = c2 * (double)f.x + (double)(Real)re;
            im = c2 * (double)f.y + (double)(Real)im;
        }
        g[i] = Cx<Real>{(Real)re, (Real)im};
    }
}

template <typename Real>
__global__ void __launch_bounds__(256) dot_kernel(DotArgs a) {
    __shared__ double red[8];
    const Cx<Real> *x = reinterpret_cast<const Cx<Real> *>(a.a);
    const Cx<Real> *y = reinterpret_cast<const Cx<Real> *>(a.b);
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    double s0 = 0.0, s1 = 0.0;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < a.nelem; i += stride) {
        const Cx<Real> p = x[i], q = y[i];
        if (a.mode == 0) {  // conj(p) q
            s0 += (double)p.x * (double)q.x + (double)p.y * (double)q.y;
            s1 += (double)p.x * (double)q.y - (double)p.y * (double)q.x;
        } else {
            const double dr = (double)p.x - a.theta * (double)q.x, di = (double)p.y - a.theta * (double)q.y;
            s0 += dr * dr + di * di;
        }
    }
    const double r0 = block_sum(s0, red);
    const double r1 = block_sum(s1, red);
    if (threadIdx.x == 0) {
        a.part[2 * blockIdx.x] = r0;
        a.part[2 * blockIdx.x + 1] = r1;
    }
}

// ---------------------------------------------------------------- launchers

static std::mutex g_krylov_lds_mu;
static std::set<const void *> g_krylov_lds_done;

static hipError_t allow_lds(const void *fn, size_t lds) {
    if (lds <= 65536) return hipSuccess;
    std::lock_guard<std::mutex> lk(g_krylov_lds_mu);
    if (g_krylov_lds_done.count(fn)) return hipSuccess;
    hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, kMaxLdsBytes);
    if (e == hipSuccess) g_krylov_lds_done.insert(fn);
    return e;
}

template <typename Real, int R, bool PF, bool SP>
static hipError_t do_ham_pf(const HamArgs &a, unsigned workers, size_t lds, hipStream_t s) {
    const void *fn = reinterpret_cast<const void *>(&ham_kernel<Real, R, PF, SP>);
    hipError_t e = allow_lds(fn, lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((ham_kernel<Real, R, PF, SP>), dim3(workers), dim3(1u << (a.geom.m - R)), lds, s, a);
    return hipGetLastError();
}

// Two register tiles fit without spilling up to 256 bytes of elements per
// thread (complex128 at R = 4 to within two registers, its first syndromes
// one mask at a time), except complex64 at R = 5, whose 32 elements per tile
// need more index and syndrome registers than the other shapes.
template <typename Real, int R>
static hipError_t do_ham(const HamArgs &a, unsigned workers, size_t lds, hipStream_t s) {
    if (a.geom.m - R < 6 || a.geom.m - R > 9) return hipErrorInvalidConfiguration;  // launch bounds
    constexpr bool pf = (2 * sizeof(Real) << R) <= 256 && !(sizeof(Real) == 4 && R == 5);
    // groups in two runs of qubits take the kernel with their address map
    if (a.geom.hi) return do_ham_pf<Real, R, pf, true>(a, workers, lds, s);
    // one tile a block (12 qubits): no next one to load, and all masks at once
    if constexpr (two_tile_limit<Real, R, pf>)
        if (1ull << a.geom.tiles_log2 <= workers) return do_ham_pf<Real, R, false, false>(a, workers, lds, s);
    return do_ham_pf<Real, R, pf, false>(a, workers, lds, s);
}

hipError_t launch_ham(bool c128, int R, const HamArgs &a, unsigned workers, size_t lds, hipStream_t s) {
    if (c128) {
        switch (R) {
            case 2: return do_ham<double, 2>(a, workers, lds, s);
            case 3: return do_ham<double, 3>(a, workers, lds, s);
            case 4: return do_ham<double, 4>(a, workers, lds, s);
            case 5: return do_ham<double, 5>(a, workers, lds, s);
        }
    } else {
        switch (R) {
            case 2: return do_ham<float, 2>(a, workers, lds, s);
            case 3: return do_ham<float, 3>(a, workers, lds, s);
            case 4: return do_ham<float, 4>(a, workers, lds, s);
            case 5: return do_ham<float, 5>(a, workers, lds, s);
        }
    }
    return hipErrorInvalidValue;
}

template <int N>
static int wave_blocks(bool high) {
    return (int)(high ? HamTile<N, true>::blocks : HamTile<N, false>::blocks);
}

int ham_wave_blocks(bool c128, int n, bool high) {
    if (!c128) return 0;
    switch (n) {
        case 16: return wave_blocks<16>(high);
        case 18: return wave_blocks<18>(high);
        case 20: return wave_blocks<20>(high);
        case 24: return wave_blocks<24>(high);
    }
    return 0;
}

template <int ROLE, int N>
static hipError_t do_ham_wave(const HamArgs &a, hipStream_t s) {
    using G = HamTile<N, ROLE == 1>;
    constexpr size_t lds = G::buf + 16 * sizeof(double);
    void (*fn)(HamArgs) = nullptr;
    if constexpr (G::wide) fn = ham_wide_kernel<ROLE>;
    else fn = ham_wave_kernel<ROLE, N>;
    hipError_t e = allow_lds(reinterpret_cast<const void *>(fn), lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(fn, dim3(G::blocks), dim3(G::T), lds, s, a);
    return hipGetLastError();
}

template <int N>
static hipError_t do_ham_role(int role, const HamArgs &a, hipStream_t s) {
    switch (role) {
        case 0: return do_ham_wave<0, N>(a, s);
        case 1: return do_ham_wave<1, N>(a, s);
        case 2: return do_ham_wave<2, N>(a, s);
        case 3: return do_ham_wave<3, N>(a, s);
        case 4: return do_ham_wave<4, N>(a, s);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_ham_wave(int role, const HamArgs &a, hipStream_t s) {
    switch (a.lat.n) {
        case 16: return do_ham_role<16>(role, a, s);
        case 18: return do_ham_role<18>(role, a, s);
        case 20: return do_ham_role<20>(role, a, s);
        case 24: return do_ham_role<24>(role, a, s);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_vec(bool c128, const VecArgs &a, unsigned blocks, hipStream_t s) {
    if (c128)
        hipLaunchKernelGGL(vec_kernel<double>, dim3(blocks), dim3(256), 0, s, a);
    else
        hipLaunchKernelGGL(vec_kernel<float>, dim3(blocks), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_scalar(const ScalarArgs &a, hipStream_t s) {
    hipLaunchKernelGGL(scalar_kernel, dim3(1), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_acc(bool c128, const AccArgs &a, unsigned blocks, hipStream_t s) {
    if (c128)
        hipLaunchKernelGGL(acc_kernel<double>, dim3(blocks), dim3(256), 0, s, a);
    else
        hipLaunchKernelGGL(acc_kernel<float>, dim3(blocks), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_dot(bool c128, const DotArgs &a, unsigned blocks, hipStream_t s) {
    if (c128)
        hipLaunchKernelGGL(dot_kernel<double>, dim3(blocks), dim3(256), 0, s, a);
    else
        hipLaunchKernelGGL(dot_kernel<float>, dim3(blocks), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_combine(bool c128, const CombineArgs &a, unsigned blocks, hipStream_t s) {
    if (c128)
        hipLaunchKernelGGL(combine_kernel<double>, dim3(blocks), dim3(256), 0, s, a);
    else
        hipLaunchKernelGGL(combine_kernel<float>, dim3(blocks), dim3(256), 0, s, a);
    return hipGetLastError();
}

}  // namespace z2h
